// HIP kernels for gfx950 (CDNA4): the fused DG right-hand side + Runge-Kutta
// stage (Sections 5.2-5.3), the period filter accumulation (Section 5.4) and
// the FP64 vector kernels of the CG iteration (Algorithm 3).
//
// Stage kernel layout: one workgroup = one 64-lane wavefront = 10 elements.
//   * the 10 x 6 x Np stage-input values are staged in LDS with coalesced
//     loads;
//   * face-node lanes compute the upwind flux (own trace from LDS, the
//     neighbour's from LDS when it belongs to the same workgroup, otherwise
//     from global memory through the connectivity code) into an LDS tile
//     laid out [face node][lane];
//   * lanes 0..59 own one (element, component) column: the reference
//     derivatives D_a y are formed with the matrix entries as wave-uniform
//     scalar operands (constant memory -> SGPRs), the two physical
//     derivatives a component contributes to the curl are exchanged between
//     the six lanes of an element with cross-lane permutes, and the lift
//     M^-1 E_f of the face fluxes is applied the same way;
//   * the RK stage update, source term, conductivity and the FP64 filter
//     accumulation run as one coalesced pass over the 10-element chunk.
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>

#include "internal.h"
#include "launch.h"
#include "mfma_cols.h"
#include "tagged.h"

namespace cmcg {

namespace {

template <int Q> struct Dim {
    static constexpr int NP = (Q + 1) * (Q + 2) * (Q + 3) / 6;
    static constexpr int NFP = (Q + 1) * (Q + 2) / 2;
};

// per-q offsets into the constant tables
__host__ __device__ constexpr int mat_size(int q) {
    return 3 * ((q + 1) * (q + 2) * (q + 3) / 6) * ((q + 1) * (q + 2) * (q + 3) / 6) +
           ((q + 1) * (q + 2) * (q + 3) / 6) * 4 * ((q + 1) * (q + 2) / 2) +
           ((q + 1) * (q + 2) * (q + 3) / 6) * ((q + 1) * (q + 2) * (q + 3) / 6);
}
__host__ __device__ constexpr int mat_off(int q) { return q <= 1 ? 0 : mat_off(q - 1) + mat_size(q - 1); }
constexpr int kMatTotal = mat_off(4);
// face-node tables as packed bytes in 32-bit words: [fnode (4 Nfp) | nnode (24 Nfp)]
__host__ __device__ constexpr int ft_words(int q) { return (28 * ((q + 1) * (q + 2) / 2) + 3) / 4; }
__host__ __device__ constexpr int ft_off(int q) { return q <= 1 ? 0 : ft_off(q - 1) + ft_words(q - 1); }
constexpr int kFtTotal = ft_off(4);

__constant__ double cMat64[kMatTotal];
__constant__ float cMat32[kMatTotal];
// Per order q, one byte per entry packed into 32-bit words: the volume node of
// face node k of face f ([f][k], 4 Nfp entries), then the volume node of the
// neighbour's face node that sits at face node k of this side, for every
// neighbour face nf and vertex permutation perm ([nf][perm][k], 24 Nfp).
__constant__ uint32_t cFaceTab[kFtTotal];

template <typename T> __device__ __forceinline__ const T* mats();
template <> __device__ __forceinline__ const double* mats<double>() { return cMat64; }
template <> __device__ __forceinline__ const float* mats<float>() { return cMat32; }

constexpr int EPW = 10;  // elements per 64-lane workgroup (60 active column lanes)

// Row access of NP contiguous values with the widest vector type the row
// alignment allows (rows start at multiples of NP * sizeof(T) bytes).
template <typename T, int NP> struct Row {
    static constexpr int BYTES = NP * (int)sizeof(T);
    static constexpr int VEC = (BYTES % 16 == 0) ? 16 : (BYTES % 8 == 0 ? 8 : (int)sizeof(T));
    static constexpr int PER = VEC / (int)sizeof(T);
    using V = typename std::conditional<VEC == 16, float4, typename std::conditional<VEC == 8, float2, T>::type>::type;
    __device__ __forceinline__ static void load(const T* __restrict__ p, T (&r)[NP]) {
        const V* q = reinterpret_cast<const V*>(p);
#pragma unroll
        for (int c = 0; c < NP / PER; ++c) {
            V v = q[c];
            const T* t = reinterpret_cast<const T*>(&v);
#pragma unroll
            for (int u = 0; u < PER; ++u) r[c * PER + u] = t[u];
        }
    }
    __device__ __forceinline__ static void store(T* __restrict__ p, const T (&r)[NP]) {
        V* q = reinterpret_cast<V*>(p);
#pragma unroll
        for (int c = 0; c < NP / PER; ++c) {
            V v;
            T* t = reinterpret_cast<T*>(&v);
#pragma unroll
            for (int u = 0; u < PER; ++u) t[u] = r[c * PER + u];
            q[c] = v;
        }
    }
};

// Low parts of a compensated FP32 state, stored as bfloat16 (8 more significant
// bits than the FP32 high part; round to nearest even).
__device__ __forceinline__ uint16_t to_bf16(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint32_t h) { return __uint_as_float(h << 16); }

// s + e == a + b exactly (Knuth's branch-free two-sum, any magnitudes).
__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e) {
    s = a + b;
    const float bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// NP bfloat16 low parts of one row (rows start at multiples of 2 NP bytes;
// NP is even for every order, so 4-byte words always line up).
template <int NP> struct RowH {
    static_assert(NP % 2 == 0, "bfloat16 rows need an even node count");
    static constexpr int PER = (2 * NP) % 8 == 0 ? 4 : 2;
    using V = typename std::conditional<PER == 4, uint2, uint32_t>::type;
    __device__ __forceinline__ static void load(const uint16_t* __restrict__ p, float (&r)[NP]) {
        const V* q = reinterpret_cast<const V*>(p);
#pragma unroll
        for (int c = 0; c < NP / PER; ++c) {
            V v = q[c];
            const uint32_t* w = reinterpret_cast<const uint32_t*>(&v);
#pragma unroll
            for (int u = 0; u < PER / 2; ++u) {
                r[c * PER + 2 * u] = from_bf16(w[u] & 0xffffu);
                r[c * PER + 2 * u + 1] = from_bf16(w[u] >> 16);
            }
        }
    }
    __device__ __forceinline__ static void store(uint16_t* __restrict__ p, const float (&r)[NP]) {
        V* q = reinterpret_cast<V*>(p);
#pragma unroll
        for (int c = 0; c < NP / PER; ++c) {
            V v;
            uint32_t* w = reinterpret_cast<uint32_t*>(&v);
#pragma unroll
            for (int u = 0; u < PER / 2; ++u)
                w[u] = (uint32_t)to_bf16(r[c * PER + 2 * u]) | ((uint32_t)to_bf16(r[c * PER + 2 * u + 1]) << 16);
            q[c] = v;
        }
    }
};

// Logical workgroup index with consecutive indices on one XCD: the hardware
// hands workgroup b to XCD b % 8, so b -> (b % 8) * per + b / 8 keeps each
// XCD on a contiguous element range (its face neighbours stay in that XCD's
// L2).  The grid is a multiple of 8; indices past the element range exit.
__device__ __forceinline__ int64_t xcd_block(int64_t per) {
    const int64_t b = blockIdx.x;
    return (b & 7) * per + (b >> 3);
}

// Arguments of this workgroup's member in a batched launch (grid.y = member):
// field, source and filter pointers move by whole members, the stage scalars
// come from the member table; returns false when the member is idle (CG
// converged, or all of its steps in this period already taken).
template <typename T>
__device__ __forceinline__ void member_offsets(const StageArgs& in, int b, StageArgs& a) {
    const double* p = in.mtab + (int64_t)b * kMemberParams;
    a.cy = p[0];
    a.ca = p[1];
    a.cu = p[2];
    a.scos = p[3];
    a.ssin = p[4];
    a.fa_re = p[5];
    a.fa_im = p[6];
    a.fb_re = p[7];
    a.fb_im = p[8];
    const int64_t fo = (int64_t)b * in.bstride;
    if (in.Y) a.Y = (const T*)in.Y + fo;
    if (in.U) a.U = (const T*)in.U + fo;
    if (in.Ynext) a.Ynext = (T*)in.Ynext + fo;
    if (in.Acc) a.Acc = (T*)in.Acc + fo;
    if (in.Uout) a.Uout = (T*)in.Uout + fo;
    if (in.Kout) a.Kout = (T*)in.Kout + fo;
    if (in.Ulo) a.Ulo = (uint16_t*)in.Ulo + fo;
    if (in.Fre) a.Fre = in.Fre + fo;
    if (in.Fim) a.Fim = in.Fim + fo;
    a.geo = (const T*)in.geo + (int64_t)b * in.gstride;
    if (in.Sre) a.Sre = (const T*)in.Sre + (int64_t)b * in.sstride;
    if (in.Sim) a.Sim = (const T*)in.Sim + (int64_t)b * in.sstride;
    if (in.smask) a.smask = in.smask + (int64_t)b * ((in.K + EPW - 1) / EPW);
}
template <typename T>
__device__ __forceinline__ bool member_args(const StageArgs& in, StageArgs& a) {
    a = in;
    if (!in.mtab) return true;
    const int b = blockIdx.y;
    if (!in.active[b]) return false;
    if (in.step >= 0 && in.step >= in.msteps[b]) return false;
    member_offsets<T>(in, b, a);
    return true;
}

// One chunk's stage input and geometry (16-byte coalesced loads, all issued
// before the first is consumed) and its connectivity codes; put() stores them
// in LDS with the stage-input rows padded to NP + 1.  NTH threads share the
// work (thread index `lane` < NTH).
template <typename T, int Q, int NTH = 64> struct ChunkIn {
    static constexpr int NP = Dim<Q>::NP;
    static constexpr int PV = 16 / (int)sizeof(T);  // values per load
    static constexpr int NY = (EPW * 6 * NP / PV + NTH - 1) / NTH, NG = (EPW * kGeo / PV + NTH - 1) / NTH;
    using V = typename std::conditional<sizeof(T) == 8, double2, float4>::type;
    static_assert((6 * NP) % PV == 0 && kGeo % PV == 0, "rows must split into 16-byte groups");
    static constexpr int NT = (ft_words(Q) + NTH - 1) / NTH;  // face-table words per thread
    V y[NY], g[NG];
    int cd;
    uint32_t tw[NT];
    __device__ __forceinline__ void fetch(const T* __restrict__ Y, const T* __restrict__ geo,
                                          const int* __restrict__ conn, int64_t e0, int ne, int lane) {
        const V* Y4 = reinterpret_cast<const V*>(Y + e0 * 6 * NP);
        const V* G4 = reinterpret_cast<const V*>(geo + e0 * kGeo);
#pragma unroll
        for (int i = 0; i < NT; ++i)
            if (lane + NTH * i < ft_words(Q)) tw[i] = cFaceTab[ft_off(Q) + lane + NTH * i];
#pragma unroll
        for (int i = 0; i < NY; ++i)
            if (lane + NTH * i < ne * 6 * NP / PV) y[i] = Y4[lane + NTH * i];
#pragma unroll
        for (int i = 0; i < NG; ++i)
            if (lane + NTH * i < ne * kGeo / PV) g[i] = G4[lane + NTH * i];
        cd = lane < ne * 4 ? conn[e0 * 4 + lane] : -3;
    }
    // keep: bit e clear stages element e's input as zero (an input mask, B P y)
    __device__ __forceinline__ void put(T* sY, T* sG, int* sC, uint8_t* sT, int ne, int lane,
                                        uint32_t keep = 0xffffffffu) const {
        uint32_t* sT4 = reinterpret_cast<uint32_t*>(sT);
#pragma unroll
        for (int i = 0; i < NT; ++i)
            if (lane + NTH * i < ft_words(Q)) sT4[lane + NTH * i] = tw[i];
#pragma unroll
        for (int i = 0; i < NY; ++i) {
            const int g4 = lane + NTH * i;
            if (g4 < ne * 6 * NP / PV) {
                const T* t = reinterpret_cast<const T*>(&y[i]);
#pragma unroll
                for (int u = 0; u < PV; ++u) {
                    const int v = PV * g4 + u;
                    sY[v + v / NP] = ((keep >> (v / (6 * NP))) & 1u) ? t[u] : T(0);
                }
            }
        }
        V* sG4 = reinterpret_cast<V*>(sG);
#pragma unroll
        for (int i = 0; i < NG; ++i)
            if (lane + NTH * i < ne * kGeo / PV) sG4[lane + NTH * i] = g[i];
        if (lane < ne * 4) sC[lane] = cd;
    }
};

// The face-node tables reach LDS with the chunk (ChunkIn): own face nodes
// [f][k], then the node of the neighbour's face seen from this side
// [nf][perm][k], one byte each.

// Flux items of a lane: item it = lane + 64 r is face node k = it / ne of
// element fe = it % ne (consecutive lanes on different elements); computed
// once per chunk (the divisor is the compile-time chunk size for full chunks).
template <int Q, int RF> struct FluxItems {
    int k[RF], fe[RF];
    bool on[RF];
    __device__ __forceinline__ void init(int ne, int lane) {
        constexpr int NFP = Dim<Q>::NFP;
#pragma unroll
        for (int r = 0; r < RF; ++r) {
            const int it = lane + 64 * r;
            on[r] = it < ne * NFP;
            const int kk = ne == EPW ? it / EPW : it / ne;
            k[r] = on[r] ? kk : 0;
            fe[r] = on[r] ? it - kk * ne : 0;
        }
    }
};

// Neighbour traces of one face for the flux items a lane owns: the
// connectivity code and the neighbour's node come from LDS.  A neighbour in
// the same chunk (about half of the interior faces of a cube-ordered mesh)
// is read from the staged tile later (loc = its LDS offset); the others are
// one round of global loads (cache-resident: neighbours are nearby in the
// element ordering).  Boundary items keep the code and build a ghost later.
template <typename T, int Q, int RF> struct TraceGather {
    static constexpr int RS = Dim<Q>::NP + 1;  // staged row stride
    T v[RF][6];
    int code[RF], loc[RF];
    // imask (nullable): input mask, one word per element block; a neighbour
    // whose bit (xor inv) is clear contributes a zero trace
    __device__ __forceinline__ void issue(const T* __restrict__ Y, const int* sC, const uint8_t* sT,
                                          const FluxItems<Q, RF>& itm, int f, int64_t e0, int ne,
                                          const uint32_t* __restrict__ imask = nullptr, int inv = 0) {
        constexpr int NP = Dim<Q>::NP, NFP = Dim<Q>::NFP;
#pragma unroll
        for (int r = 0; r < RF; ++r) {
            code[r] = -3;
            loc[r] = -1;
            if (itm.on[r]) {
                const int cd = sC[itm.fe[r] * 4 + f];
                code[r] = cd;
                if (cd >= 0) {
                    const int nn = sT[4 * NFP + (((cd >> 3) & 3) * 6 + (cd & 7)) * NFP + itm.k[r]];
                    const int64_t nb = cd >> 5;
                    const int64_t d = nb - e0;
                    if (d >= 0 && d < ne) {
                        loc[r] = (int)d * 6 * RS + nn;
                    } else if (imask && !(((imask[nb / EPW] >> (int)(nb % EPW)) & 1u) ^ (uint32_t)inv)) {
#pragma unroll
                        for (int cc = 0; cc < 6; ++cc) v[r][cc] = T(0);
                    } else {
                        const T* q = Y + nb * 6 * NP + nn;
#pragma unroll
                        for (int cc = 0; cc < 6; ++cc) v[r][cc] = q[cc * NP];
                    }
                }
            }
        }
    }
    // neighbour values of item r (after issue; sY = the staged chunk)
    __device__ __forceinline__ void values(const T* sY, int r, T (&Ep)[3], T (&Hp)[3]) const {
        if (loc[r] >= 0) {
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                Ep[cc] = sY[loc[r] + cc * RS];
                Hp[cc] = sY[loc[r] + (3 + cc) * RS];
            }
        } else {
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                Ep[cc] = v[r][cc];
                Hp[cc] = v[r][3 + cc];
            }
        }
    }
};

// Arithmetic that the stage and the period kernels share is written with
// explicit fma(): left to the compiler, they may contract the same expression
// differently, and their results would part in the last bit.
//
// Upwind flux (E, then H rows) at one face node, g = the face's normal and
// flux coefficients.
template <typename T>
__device__ __forceinline__ void upwind3(const T* g, const T (&Em)[3], const T (&Hm)[3], const T (&Ep)[3],
                                        const T (&Hp)[3], T (&o)[6]) {
    const T n0 = g[0], n1 = g[1], n2 = g[2];
    const T cE1 = g[3], cE2 = g[4], cH1 = g[5], cH2 = g[6];
    const T dE0 = Ep[0] - Em[0], dE1 = Ep[1] - Em[1], dE2 = Ep[2] - Em[2];
    const T dH0 = Hp[0] - Hm[0], dH1 = Hp[1] - Hm[1], dH2 = Hp[2] - Hm[2];
    const T ndE = fma(n0, dE0, fma(n1, dE1, n2 * dE2));
    const T ndH = fma(n0, dH0, fma(n1, dH1, n2 * dH2));
    o[0] = fma(cE1, fma(-ndE, n0, dE0), -cE2 * fma(n1, dH2, -n2 * dH1));
    o[1] = fma(cE1, fma(-ndE, n1, dE1), -cE2 * fma(n2, dH0, -n0 * dH2));
    o[2] = fma(cE1, fma(-ndE, n2, dE2), -cE2 * fma(n0, dH1, -n1 * dH0));
    o[3] = fma(cH1, fma(-ndH, n0, dH0), cH2 * fma(n1, dE2, -n2 * dE1));
    o[4] = fma(cH1, fma(-ndH, n1, dH1), cH2 * fma(n2, dE0, -n0 * dE2));
    o[5] = fma(cH1, fma(-ndH, n2, dH2), cH2 * fma(n0, dE1, -n1 * dE0));
}

// PIPE: request the next face's neighbour traces (and, before the last face,
// the update operands) one face ahead.  Without it every face gathers and
// consumes in turn, which needs fewer registers.
// MH: several-frequency problems (further source harmonics and filters);
// the single-frequency instantiation carries none of that code.
// LTSM: the local-time-stepping substep modes (LTS_FWD, LTS_ADJ) only.
template <typename T, int Q, bool PIPE, bool MH, bool LTSM = false>
__global__ __launch_bounds__(64) void k_stage(StageArgs args, int64_t per) {
    constexpr int NP = Dim<Q>::NP, NFP = Dim<Q>::NFP, NF4 = 4 * NFP;
    constexpr int RS = NP + 1;            // padded LDS row stride (bank spread)
    constexpr int MO = mat_off(Q);
    constexpr int LO = MO + 3 * NP * NP;  // LIFT [NP][NF4]
    constexpr int RF = (EPW * NFP + 63) / 64;  // flux items per lane and face
    constexpr int FS = 65;                     // flux tile row stride (bank spread)
    __shared__ T sY[EPW * 6 * RS];
    __shared__ T sF[NFP * FS];
    __shared__ T sG[EPW * kGeo];
    __shared__ int sC[EPW * 4];
    __shared__ __align__(4) uint8_t sT[4 * ft_words(Q)];

    StageArgs a;
    if (!member_args<T>(args, a)) return;  // uniform per workgroup
    int64_t blk = xcd_block(per);
    if (a.blist) {  // only the listed element blocks
        if (blk >= a.nblist) return;
        blk = a.blist[blk];
    }
    const int64_t e0 = blk * EPW;
    if (e0 >= a.K) return;
    const T* __restrict__ Y = (const T*)a.Y;
    const int lane = threadIdx.x;
    const int ne = (int)((a.K - e0) < EPW ? (a.K - e0) : EPW);
    const int64_t base = e0 * 6 * NP;

    // column ownership: lane = (element, component)
    const int el = lane / 6;
    const int c = lane - 6 * el;
    const bool act = el < ne;
    const int elc = act ? el : 0;
    const int row = elc * 6 + c;
    const int64_t grow = base + (int64_t)row * NP;
    const int mode = a.mode;
    constexpr bool COMP = std::is_same<T, float>::value;  // compensated state U + Ulo
    const bool needL = COMP && (mode == RK2_S2 || mode == RK4_S4);
    const bool needU =
        LTSM ? (mode == LTS_FWD || mode == LTS_ADJ) : (mode == RK2_S2 || mode == RK4_S2 || mode == RK4_S3 || needL);
    const bool needA = LTSM ? (mode == LTS_ADJ || (mode == LTS_FWD && a.Acc != nullptr))
                            : (mode == RK4_S2 || mode == RK4_S3 || mode == RK4_S4);

    const uint32_t keep = a.imask ? (a.imask[blk] ^ (a.imask_inv ? 0xffffffffu : 0u)) : 0xffffffffu;
    {
        ChunkIn<T, Q> in;
        in.fetch(Y, (const T*)a.geo, a.conn, e0, ne, lane);
        in.put(sY, sG, sC, sT, ne, lane, keep);
    }
    __syncthreads();
    // neighbour traces of face 0 in flight during the volume work
    FluxItems<Q, RF> itm;
    itm.init(ne, lane);
    TraceGather<T, Q, RF> cur, nxt;
    if (PIPE) cur.issue(Y, sC, sT, itm, 0, e0, ne, a.imask, a.imask_inv);

    // ---- volume term: D_a y per column, curl terms exchanged between lanes
    T y[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) y[j] = sY[row * RS + j];
    const T* gg = &sG[elc * kGeo];
    const int c3 = c < 3 ? c : c - 3;
    const int kp = c3 == 0 ? 2 : c3 - 1;  // (c3 + 2) % 3
    const int km = c3 == 2 ? 0 : c3 + 1;  // (c3 + 1) % 3
    const int sb = elc * 6 + (c < 3 ? 3 : 0);
    const int lane_p = sb + (c3 == 0 ? 2 : c3 - 1);  // sends +d_{m+1} V_{m+2} (m = c3)
    const int lane_m = sb + (c3 == 2 ? 0 : c3 + 1);  // sends -d_{m+2} V_{m+1}
    const T* Mt = mats<T>();
    // this column's contributions to the curl of its field:
    // pv = d_{c3+2} V_{c3} (to curl component c3+1), mv = -d_{c3+1} V_{c3} (to c3+2)
    T pv[NP], mv[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        pv[i] = T(0);
        mv[i] = T(0);
    }
#pragma unroll 1
    for (int ax = 0; ax < 3; ++ax) {
        const T gp = gg[3 * ax + kp];
        const T gm = gg[3 * ax + km];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            T d = T(0);
#pragma unroll
            for (int j = 0; j < NP; ++j) d = fma(Mt[MO + (ax * NP + i) * NP + j], y[j], d);
            pv[i] = fma(gp, d, pv[i]);
            mv[i] = fma(-gm, d, mv[i]);
        }
    }
    // E rows take -curl H, H rows +curl E
    const T sgn = c < 3 ? T(-1) : T(1);
    T acc[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) acc[i] = sgn * (__shfl(pv[i], lane_p) + __shfl(mv[i], lane_m));

    // ---- upwind flux and lift, one face at a time; the next face's
    // neighbour traces (and before the last face the update operands) are
    // requested before this face's work
    T up[NP], ap[NP];
    float lo[NP];
#pragma unroll 1
    for (int f = 0; f < 4; ++f) {
        if (PIPE) {
            if (f < 3) {
                nxt.issue(Y, sC, sT, itm, f + 1, e0, ne, a.imask, a.imask_inv);
            } else if (act) {
                if (needU) Row<T, NP>::load((const T*)a.U + grow, up);
                if (needA) Row<T, NP>::load((const T*)a.Acc + grow, ap);
                if constexpr (COMP)
                    if (needL) RowH<NP>::load((const uint16_t*)a.Ulo + grow, lo);
            }
        } else {
            cur.issue(Y, sC, sT, itm, f, e0, ne, a.imask, a.imask_inv);
        }
#pragma unroll
        for (int r = 0; r < RF; ++r) {
            if (!itm.on[r]) continue;
            const int k = itm.k[r];
            const int fe = itm.fe[r];
            const int own = sT[f * NFP + k];
            T Em[3], Hm[3], Ep[3], Hp[3];
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                Em[cc] = sY[(fe * 6 + cc) * RS + own];
                Hm[cc] = sY[(fe * 6 + 3 + cc) * RS + own];
            }
            const int code = cur.code[r];
            if (code >= 0) {
                cur.values(sY, r, Ep, Hp);
            } else if (code == -1) {  // PEC ghost: E+ = -E-, H+ = H-
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    Ep[cc] = -Em[cc];
                    Hp[cc] = Hm[cc];
                }
            } else {  // impedance ghost (homogeneous part): zero exterior state
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    Ep[cc] = T(0);
                    Hp[cc] = T(0);
                }
            }
            T fx[6];
            upwind3(&sG[fe * kGeo + 9 + 7 * f], Em, Hm, Ep, Hp, fx);
            T* o = &sF[k * FS + fe * 6];
#pragma unroll
            for (int cc = 0; cc < 6; ++cc) o[cc] = fx[cc];
        }
        __syncthreads();
        T fl[NFP];
#pragma unroll
        for (int k = 0; k < NFP; ++k) fl[k] = sF[k * FS + lane];
        __syncthreads();  // the tile is rewritten by the next face
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            T s = acc[i];
#pragma unroll
            for (int k = 0; k < NFP; ++k) s = fma(Mt[LO + i * NF4 + f * NFP + k], fl[k], s);
            acc[i] = s;
        }
        if (PIPE && f < 3) cur = nxt;
    }
    if (!act) return;
    if (!PIPE) {
        if (needU) Row<T, NP>::load((const T*)a.U + grow, up);
        if (needA) Row<T, NP>::load((const T*)a.Acc + grow, ap);
        if constexpr (COMP)
            if (needL) RowH<NP>::load((const uint16_t*)a.Ulo + grow, lo);
    }

    // ---- stage update on the lane's row
    const T inv = c < 3 ? gg[37] : gg[38];
    const T sig = c < 3 ? gg[39] : T(0);
    T kv[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) kv[i] = fma(inv, acc[i], -sig * y[i]);
    if (c < a.src_rows && (!a.smask || ((a.smask[blk] >> elc) & 1u))) {
        T sr[NP], si[NP];
        Row<T, NP>::load((const T*)a.Sre + grow, sr);
        Row<T, NP>::load((const T*)a.Sim + grow, si);
        const T scos = (T)a.scos, ssin = (T)a.ssin;
#pragma unroll
        for (int i = 0; i < NP; ++i) kv[i] = fma(scos, sr[i], fma(-ssin, si[i], kv[i]));
#pragma unroll 1
        // further harmonics of a several-frequency source (single launches, so the
        // kernel arguments hold the tables; indexing the local copy put it in scratch)
        for (int h = 1; MH && h < a.nharm; ++h) {
            Row<T, NP>::load((const T*)args.Sre + h * args.hstride + grow, sr);
            Row<T, NP>::load((const T*)args.Sim + h * args.hstride + grow, si);
            const T hc = (T)args.hcos[h], hs = (T)args.hsin[h];
#pragma unroll
            for (int i = 0; i < NP; ++i) kv[i] += hc * sr[i] - hs * si[i];
        }
    }
    const T cy = (T)a.cy, ca = (T)a.ca, cu = (T)a.cu;
    T o1[NP], o2[NP];
    if constexpr (LTSM) {
        if (mode == LTS_CHAIN) {
            auto on = [&](const uint32_t* m, int inv) {
                return !m || ((((m[blk] >> elc) & 1u) ^ (uint32_t)inv) != 0);
            };
            const bool oa = on(a.lmask, a.linv), ob = on(a.lmaskB, a.linvB), oc = on(a.lmaskC, a.linvC);
#pragma unroll
            for (int i = 0; i < NP; ++i) o1[i] = oa ? kv[i] : T(0);
            T x[NP];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const bool use = j == 0 ? ob : j == 1 ? oc : true;
                if (!args.lw[j] || !use) continue;
                Row<T, NP>::load((const T*)args.lw[j] + grow, x);
#pragma unroll
                for (int i = 0; i < NP; ++i) o1[i] += x[i];
            }
            Row<T, NP>::store((T*)a.Uout + grow, o1);
        } else if (mode == LTS_FWD) {
            T w[NP];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j >= a.lnw) break;
                Row<T, NP>::load((const T*)args.lw[j] + grow, w);
                const T cj = (T)args.lcw[j];
#pragma unroll
                for (int i = 0; i < NP; ++i) kv[i] = fma(cj, w[i], kv[i]);
            }
            const T le = (T)a.le, lf = (T)a.lf;
            const bool hasA = a.Acc != nullptr;
            if (a.Ynext) {
#pragma unroll
                for (int i = 0; i < NP; ++i) o1[i] = fma(cy, kv[i], hasA ? fma(le, ap[i], up[i]) : up[i]);
                Row<T, NP>::store((T*)a.Ynext + grow, o1);
            }
            if (a.Uout) {
#pragma unroll
                for (int i = 0; i < NP; ++i) o2[i] = hasA ? fma(ca, kv[i], lf * ap[i]) : ca * kv[i];
                Row<T, NP>::store((T*)a.Uout + grow, o2);
            }
        } else {
            const bool on = ((a.lmask[blk] >> elc) & 1u) != 0;
            if (on) {
                T w[NP];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (j >= a.lnw) break;
                    T* wj = (T*)args.lw[j] + grow;
                    if (a.linit) {
#pragma unroll
                        for (int i = 0; i < NP; ++i) w[i] = T(0);
                    } else {
                        Row<T, NP>::load(wj, w);
                    }
                    const T cj = (T)args.lcw[j];
#pragma unroll
                    for (int i = 0; i < NP; ++i) w[i] = fma(cj, y[i], w[i]);
                    Row<T, NP>::store(wj, w);
                }
            }
            const T le = (T)a.le, lf = (T)a.lf;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const T A = on ? kv[i] : T(0);
                o1[i] = up[i] + A;
                o2[i] = fma(lf, A, le * ap[i]);
            }
            Row<T, NP>::store((T*)a.Uout + grow, o1);
            if (a.Ynext) Row<T, NP>::store((T*)a.Ynext + grow, o2);
            if (a.lz) {  // the next substep's starting state and first stage vector
                Row<T, NP>::store((T*)a.lz + grow, o1);
                const T kc = (T)a.lkc;
#pragma unroll
                for (int i = 0; i < NP; ++i) o2[i] = kc * o1[i];
                Row<T, NP>::store((T*)a.lk + grow, o2);
            }
        }
    } else {
        switch (mode) {
            case RK2_S1:
#pragma unroll
                for (int i = 0; i < NP; ++i) o1[i] = fma(cy, kv[i], y[i]);
                Row<T, NP>::store((T*)a.Ynext + grow, o1);
                break;
            case RK2_S2:
                if constexpr (COMP) {
                    float e[NP];
#pragma unroll
                    for (int i = 0; i < NP; ++i) two_sum(up[i], fma(cu, kv[i], lo[i]), o1[i], e[i]);
                    Row<T, NP>::store((T*)a.Uout + grow, o1);
                    RowH<NP>::store((uint16_t*)a.Ulo + grow, e);
                } else {
#pragma unroll
                    for (int i = 0; i < NP; ++i) o1[i] = fma(cu, kv[i], up[i]);
                    Row<T, NP>::store((T*)a.Uout + grow, o1);
                }
                break;
            case RK4_S1:
#pragma unroll
                for (int i = 0; i < NP; ++i) {
                    o1[i] = fma(cy, kv[i], y[i]);
                    o2[i] = COMP ? ca * kv[i] : fma(ca, kv[i], y[i]);
                }
                Row<T, NP>::store((T*)a.Ynext + grow, o1);
                Row<T, NP>::store((T*)a.Acc + grow, o2);
                break;
            case RK4_S2:
            case RK4_S3:
#pragma unroll
                for (int i = 0; i < NP; ++i) {
                    o1[i] = fma(cy, kv[i], up[i]);
                    o2[i] = fma(ca, kv[i], ap[i]);
                }
                Row<T, NP>::store((T*)a.Ynext + grow, o1);
                Row<T, NP>::store((T*)a.Acc + grow, o2);
                break;
            case RK4_S4:
                if constexpr (COMP) {
                    float e[NP];
#pragma unroll
                    for (int i = 0; i < NP; ++i) two_sum(up[i], fma(cu, kv[i], ap[i]) + lo[i], o1[i], e[i]);
                    Row<T, NP>::store((T*)a.Uout + grow, o1);
                    RowH<NP>::store((uint16_t*)a.Ulo + grow, e);
                } else {
#pragma unroll
                    for (int i = 0; i < NP; ++i) o1[i] = fma(cu, kv[i], ap[i]);
                    Row<T, NP>::store((T*)a.Uout + grow, o1);
                }
                break;
            default:
                Row<T, NP>::store((T*)a.Kout + grow, kv);
                break;
        }
    }
    if (a.filter) {
        // F += fa * U + fb * k on the lane's row (U is the stage input here)
        double* fr = a.Fre + grow;
        double* fi = a.Fim + grow;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const double ud = (double)y[i], kd = (double)kv[i];
            fr[i] = fma(a.fa_re, ud, fma(a.fb_re, kd, fr[i]));
            fi[i] = fma(a.fa_im, ud, fma(a.fb_im, kd, fi[i]));
        }
#pragma unroll 1
        for (int h = 1; MH && h < a.nharm; ++h) {
            double* hr = args.Fre + h * args.hstride + grow;
            double* hi = args.Fim + h * args.hstride + grow;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const double ud = (double)y[i], kd = (double)kv[i];
                hr[i] += args.hfa_re[h] * ud + args.hfb_re[h] * kd;
                hi[i] += args.hfa_im[h] * ud + args.hfb_im[h] * kd;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// One 16x16x4 matrix-core product D = A B + C in the field precision:
// v_mfma_f32_16x16x4f32 or v_mfma_f64_16x16x4f64.  Both take A[l % 16][l / 16]
// and B[l / 16][l % 16] from lane l; their accumulators differ: register r of
// lane l holds D[row(l / 16, r)][l % 16] with row = 4 (l / 16) + r for FP32
// and 4 r + l / 16 for FP64 (measured with one-hot operands; checked against
// numpy through cmcg_debug_mfma).
template <typename T> struct Mfma;
template <> struct Mfma<float> {
    typedef float acc_t __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc_t mma(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int q4, int r) { return 4 * q4 + r; }
};
template <> struct Mfma<double> {
    typedef double acc_t __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int q4, int r) { return 4 * r + q4; }
};

// 8- and 16-byte accesses of the update pass, with the non-temporal hint where
// STREAM says so (stream_hints below; a template argument, since the compiler
// merges two branches that differ in the hint alone, and drops it).
template <typename V> struct Raw {
    typedef unsigned int W __attribute__((ext_vector_type(sizeof(V) / 4)));
};
template <bool STREAM, typename V> __device__ __forceinline__ V ldg(const void* p) {
    const auto* q = reinterpret_cast<const typename Raw<V>::W*>(p);
    if constexpr (STREAM) return __builtin_bit_cast(V, __builtin_nontemporal_load(q));
    return __builtin_bit_cast(V, *q);
}
template <bool STREAM, typename V> __device__ __forceinline__ void stg(void* p, const V& v) {
    auto* q = reinterpret_cast<typename Raw<V>::W*>(p);
    const auto w = __builtin_bit_cast(typename Raw<V>::W, v);
    if constexpr (STREAM)
        __builtin_nontemporal_store(w, q);
    else
        *q = w;
}

// Operands of the coalesced update pass (16-byte groups v = lane + NTH t of
// the chunk: 4 FP32 or 2 FP64 values), all requested before the pass
// computes: r0 = U (modes that combine with the state) or the stage input
// (stage-1 modes, filter), r1 = Acc, r2 = the bfloat16 low parts (FP32).
template <typename T, int Q, int NTH, bool LTSM, int STREAM> struct MfmaUpdateIn {
    static constexpr int PV = 16 / (int)sizeof(T);
    static constexpr bool COMP = std::is_same<T, float>::value;  // compensated state U + Ulo
    using V = typename std::conditional<COMP, float4, double2>::type;
    static constexpr int NIT = (EPW * 6 * Dim<Q>::NP / PV + NTH - 1) / NTH;
    V r0[NIT], r1[NIT];
    uint2 r2[COMP ? NIT : 1];
    V w[LTSM ? NIT : 1][4], z[LTSM ? NIT : 1];  // local time stepping: W_j, and LTS_ADJ's zbar
    __device__ __forceinline__ void fetch(const StageArgs& a, int64_t base, int nvv, int lane) {
        const int mode = a.mode;
        // LTS_FWD reads U (and Acc when given), LTS_ADJ the stage input and Acc
        const bool s1 = LTSM ? mode == LTS_ADJ : mode == RK2_S1 || mode == RK4_S1 || (mode == RHS && a.filter);
        // FP64 stage 4 forms U = Acc + cu k without the state
        const bool needU =
            LTSM ? mode == LTS_FWD : mode == RK2_S2 || mode == RK4_S2 || mode == RK4_S3 || (COMP && mode == RK4_S4);
        const bool needA = LTSM ? (mode == LTS_ADJ || (mode == LTS_FWD && a.Acc != nullptr))
                                : (mode == RK4_S2 || mode == RK4_S3 || mode == RK4_S4);
        const bool needL = !LTSM && COMP && (mode == RK2_S2 || mode == RK4_S4);
        const T* src0 = needU ? (const T*)a.U : (const T*)a.Y;
#pragma unroll
        for (int t = 0; t < NIT; ++t) {
            const int vv = lane + NTH * t;
            if (vv >= nvv) continue;
            const int64_t gi = base + PV * vv;
            if (s1 || needU) r0[t] = ldg<STREAM == 2, V>(src0 + gi);
            if (needA) r1[t] = ldg<STREAM == 2, V>((const T*)a.Acc + gi);
            if constexpr (LTSM) {
                // all at once: behind one another, at the end, they added up to
                // four memory latencies to every substep launch (P2 FP64, 12960
                // tets, four substeps: 107.1 ms a solve against 104.2)
                if (mode != LTS_CHAIN && !(mode == LTS_ADJ && a.linit)) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (j < a.lnw) w[t][j] = *reinterpret_cast<const V*>((const T*)a.lw[j] + gi);
                }
                if (mode == LTS_ADJ) z[t] = *reinterpret_cast<const V*>((const T*)a.U + gi);
            }
            if constexpr (COMP)
                if (needL) r2[t] = ldg<STREAM == 2, uint2>((const uint16_t*)a.Ulo + gi);
        }
    }
};

// Stage update of a block: one coalesced pass over its contiguous rows
// (16-byte groups v = PV (tid + NTH t)), kvals(v, kv) giving the scaled
// right-hand side of a group and upd its operands.
template <typename T, int Q, int NTH, bool MH, bool LTSM, int STREAM, typename KV>
__device__ __forceinline__ void stage_update(const StageArgs& args, const StageArgs& a,
                                             const MfmaUpdateIn<T, Q, NTH, LTSM, STREAM>& upd, int64_t blk, int64_t base,
                                             int nvv, int tid, KV kvals) {
    constexpr bool COMP = std::is_same<T, float>::value;  // compensated state U + Ulo
    constexpr int NP = Dim<Q>::NP, PV = 16 / (int)sizeof(T);
    using UIn = MfmaUpdateIn<T, Q, NTH, LTSM, STREAM>;
    using V = typename UIn::V;
    const int mode = a.mode;
    const T scos = (T)a.scos, ssin = (T)a.ssin;
    const T cy = (T)a.cy, ca = (T)a.ca, cu = (T)a.cu;
    // elements whose source is zero (and H rows of an interior source) read none
    const uint32_t sm = a.smask ? a.smask[blk] : 0xffffffffu;
    auto takes_src = [&](int row) { return row - 6 * (row / 6) < a.src_rows && ((sm >> (row / 6)) & 1u); };
    auto ldv = [](const void* p, int64_t o, T (&r)[PV]) {
        const V v = *reinterpret_cast<const V*>((const T*)p + o);
        const T* t = reinterpret_cast<const T*>(&v);
#pragma unroll
        for (int u = 0; u < PV; ++u) r[u] = t[u];
    };
#pragma unroll
    for (int t = 0; t < UIn::NIT; ++t) {
        const int vv = tid + NTH * t;
        if (vv >= nvv) continue;
        const int v = PV * vv;
        const int64_t gi = base + v;
        T kv[PV];
        kvals(v, kv);
        if (a.src_rows > 0 && (takes_src(v / NP) || takes_src((v + PV - 1) / NP))) {
            T srv[PV], siv[PV];
            ldv(a.Sre, gi, srv);
            ldv(a.Sim, gi, siv);
#pragma unroll
            for (int u = 0; u < PV; ++u) {
                const int row = (v + u) / NP;
                if (takes_src(row)) kv[u] = fma(scos, srv[u], fma(-ssin, siv[u], kv[u]));
            }
#pragma unroll 1
            // further harmonics (tables read from the kernel arguments, as in k_stage)
            for (int h = 1; MH && h < a.nharm; ++h) {
                T hrv[PV], hiv[PV];
                ldv(args.Sre, h * args.hstride + gi, hrv);
                ldv(args.Sim, h * args.hstride + gi, hiv);
                const T hc = (T)args.hcos[h], hs = (T)args.hsin[h];
#pragma unroll
                for (int u = 0; u < PV; ++u) {
                    const int row = (v + u) / NP;
                    if (takes_src(row)) kv[u] += hc * hrv[u] - hs * hiv[u];
                }
            }
        }
        T x0[PV], x1[PV];  // U (or Y in stage-1 modes), Acc
        {
            const T* p0 = reinterpret_cast<const T*>(&upd.r0[t]);
            const T* p1 = reinterpret_cast<const T*>(&upd.r1[t]);
#pragma unroll
            for (int u = 0; u < PV; ++u) {
                x0[u] = p0[u];
                x1[u] = p1[u];
            }
        }
        T lo[PV];
        if constexpr (COMP) {
            if (mode == RK2_S2 || mode == RK4_S4) {
                lo[0] = from_bf16(upd.r2[t].x & 0xffffu);
                lo[1] = from_bf16(upd.r2[t].x >> 16);
                lo[2] = from_bf16(upd.r2[t].y & 0xffffu);
                lo[3] = from_bf16(upd.r2[t].y >> 16);
            }
        }
        auto stv = [&](void* p, const T (&o)[PV]) {
            V w;
            T* q = reinterpret_cast<T*>(&w);
#pragma unroll
            for (int u = 0; u < PV; ++u) q[u] = o[u];
            stg<STREAM == 2, V>((T*)p + gi, w);
        };
        T o1[PV], o2[PV];
        if constexpr (LTSM) {
            if (mode == LTS_CHAIN) {
                const int el = v / NP / 6;  // a 16-byte group never straddles an element
                auto on = [&](const uint32_t* m, int inv) {
                    return !m || ((((m[blk] >> el) & 1u) ^ (uint32_t)inv) != 0);
                };
                const bool oa = on(a.lmask, a.linv), ob = on(a.lmaskB, a.linvB), oc = on(a.lmaskC, a.linvC);
#pragma unroll
                for (int u = 0; u < PV; ++u) o1[u] = oa ? kv[u] : T(0);
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    const bool use = j == 0 ? ob : j == 1 ? oc : true;
                    if (!args.lw[j] || !use) continue;
                    T x[PV];
                    ldv(args.lw[j], gi, x);
#pragma unroll
                    for (int u = 0; u < PV; ++u) o1[u] += x[u];
                }
                stv(a.Uout, o1);
            } else if (mode == LTS_FWD) {  // x0 = U, x1 = Acc
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (j >= a.lnw) break;
                    const T* w = reinterpret_cast<const T*>(&upd.w[t][j]);
                    const T cj = (T)args.lcw[j];
#pragma unroll
                    for (int u = 0; u < PV; ++u) kv[u] = fma(cj, w[u], kv[u]);
                }
                const T le = (T)a.le, lf = (T)a.lf;
                const bool hasA = a.Acc != nullptr;
                if (a.Ynext) {
#pragma unroll
                    for (int u = 0; u < PV; ++u) o1[u] = fma(cy, kv[u], hasA ? fma(le, x1[u], x0[u]) : x0[u]);
                    stv(a.Ynext, o1);
                }
                if (a.Uout) {
#pragma unroll
                    for (int u = 0; u < PV; ++u) o2[u] = hasA ? fma(ca, kv[u], lf * x1[u]) : ca * kv[u];
                    stv(a.Uout, o2);
                }
            } else {  // x0 = the stage input kcur, x1 = Acc
                // a 16-byte group never straddles an element (6 NP is a multiple of 4)
                const bool on = ((a.lmask[blk] >> (v / NP / 6)) & 1u) != 0;
                if (on) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (j >= a.lnw) break;
                        T w[PV];
                        if (a.linit) {
#pragma unroll
                            for (int u = 0; u < PV; ++u) w[u] = T(0);
                        } else {
                            const T* wj = reinterpret_cast<const T*>(&upd.w[t][j]);
#pragma unroll
                            for (int u = 0; u < PV; ++u) w[u] = wj[u];
                        }
                        const T cj = (T)args.lcw[j];
#pragma unroll
                        for (int u = 0; u < PV; ++u) w[u] = fma(cj, x0[u], w[u]);
                        stv(const_cast<void*>(args.lw[j]), w);
                    }
                }
                const T* z = reinterpret_cast<const T*>(&upd.z[t]);
                const T le = (T)a.le, lf = (T)a.lf;
#pragma unroll
                for (int u = 0; u < PV; ++u) {
                    const T A = on ? kv[u] : T(0);
                    o1[u] = z[u] + A;
                    o2[u] = fma(lf, A, le * x1[u]);
                }
                stv(a.Uout, o1);
                if (a.Ynext) stv(a.Ynext, o2);
                if (a.lz) {  // the next substep's starting state and first stage vector
                    stv(a.lz, o1);
                    const T kc = (T)a.lkc;
#pragma unroll
                    for (int u = 0; u < PV; ++u) o2[u] = kc * o1[u];
                    stv(a.lk, o2);
                }
            }
        } else {
            switch (mode) {
                case RK2_S1:
#pragma unroll
                    for (int u = 0; u < PV; ++u) o1[u] = fma(cy, kv[u], x0[u]);
                    stv(a.Ynext, o1);
                    break;
                case RK2_S2:
                    if constexpr (COMP) {
#pragma unroll
                        for (int u = 0; u < PV; ++u) two_sum(x0[u], fma(cu, kv[u], lo[u]), o1[u], o2[u]);
                        stv(a.Uout, o1);
                        uint2 w;
                        w.x = (uint32_t)to_bf16(o2[0]) | ((uint32_t)to_bf16(o2[1]) << 16);
                        w.y = (uint32_t)to_bf16(o2[2]) | ((uint32_t)to_bf16(o2[3]) << 16);
                        stg<STREAM == 2, uint2>((uint16_t*)a.Ulo + gi, w);
                    } else {
#pragma unroll
                        for (int u = 0; u < PV; ++u) o1[u] = fma(cu, kv[u], x0[u]);
                        stv(a.Uout, o1);
                    }
                    break;
                case RK4_S1:
#pragma unroll
                    for (int u = 0; u < PV; ++u) {
                        o1[u] = fma(cy, kv[u], x0[u]);
                        o2[u] = COMP ? ca * kv[u] : fma(ca, kv[u], x0[u]);
                    }
                    stv(a.Ynext, o1);
                    stv(a.Acc, o2);
                    break;
                case RK4_S2:
                case RK4_S3:
#pragma unroll
                    for (int u = 0; u < PV; ++u) {
                        o1[u] = fma(cy, kv[u], x0[u]);
                        o2[u] = fma(ca, kv[u], x1[u]);
                    }
                    stv(a.Ynext, o1);
                    stv(a.Acc, o2);
                    break;
                case RK4_S4:
                    if constexpr (COMP) {
#pragma unroll
                        for (int u = 0; u < PV; ++u) two_sum(x0[u], fma(cu, kv[u], x1[u]) + lo[u], o1[u], o2[u]);
                        stv(a.Uout, o1);
                        uint2 w;
                        w.x = (uint32_t)to_bf16(o2[0]) | ((uint32_t)to_bf16(o2[1]) << 16);
                        w.y = (uint32_t)to_bf16(o2[2]) | ((uint32_t)to_bf16(o2[3]) << 16);
                        stg<STREAM == 2, uint2>((uint16_t*)a.Ulo + gi, w);
                    } else {
#pragma unroll
                        for (int u = 0; u < PV; ++u) o1[u] = fma(cu, kv[u], x1[u]);
                        stv(a.Uout, o1);
                    }
                    break;
                default:
                    stv(a.Kout, kv);
                    break;
            }
        }
        if (a.filter) {  // stage-1 and RHS modes: x0 is the stage input
            double2 fr[PV / 2], fi[PV / 2];
#pragma unroll
            for (int u = 0; u < PV / 2; ++u) {
                fr[u] = ldg<STREAM != 0, double2>(a.Fre + gi + 2 * u);
                fi[u] = ldg<STREAM != 0, double2>(a.Fim + gi + 2 * u);
            }
#pragma unroll
            for (int u = 0; u < PV; ++u) {
                const double ud = (double)x0[u], kd = (double)kv[u];
                double& re = u % 2 ? fr[u / 2].y : fr[u / 2].x;
                double& im = u % 2 ? fi[u / 2].y : fi[u / 2].x;
                re = fma(a.fa_re, ud, fma(a.fb_re, kd, re));
                im = fma(a.fa_im, ud, fma(a.fb_im, kd, im));
            }
#pragma unroll
            for (int u = 0; u < PV / 2; ++u) {
                stg<STREAM != 0, double2>(a.Fre + gi + 2 * u, fr[u]);
                stg<STREAM != 0, double2>(a.Fim + gi + 2 * u, fi[u]);
            }
#pragma unroll 1
            for (int h = 1; MH && h < a.nharm; ++h)
#pragma unroll
                for (int u = 0; u < PV; ++u) {
                    const double ud = (double)x0[u], kd = (double)kv[u];
                    args.Fre[h * args.hstride + gi + u] += args.hfa_re[h] * ud + args.hfb_re[h] * kd;
                    args.Fim[h * args.hstride + gi + u] += args.hfa_im[h] * ud + args.hfb_im[h] * kd;
                }
        }
    }
}

// ---------------------------------------------------------------------------
// FP64 stage kernel on the matrix cores (q = 2, 3).
//
// Columns n = element * 6 + s of a block of 10 elements; wave w of four owns the
// column tile 16 w .. 16 w + 15 and all its rows:
//   volume:  C[i][n] = sum_{a,j} D_a[i][j] W_a[j][n],  W_a = sgn (grad xi_a x V)_m,
//            V = H for s < 3 (E rows, sgn = -1), V = E for s >= 3 (sgn = +1),
//            m = s mod 3 -- i.e. curl V = sum_a D_a (grad xi_a x V) for an affine
//            element, so the product already is the curl column;
//   lift:    C[i][n] += sum_{f,k} LIFT[i][f Nfp + k] flux[f][k][n], all faces.
// Rows 0 .. 15 run on v_mfma_f64_16x16x4, P3's rows 16 .. 19 on
// v_mfma_f64_4x4x4_4b, whose four blocks are the tile's four groups of four
// columns: both take B[l / 16][l % 16] from lane l, so an operand is built once
// and no row of P3 is padded (a second 16-row tile would spend 12 of its 16 rows
// on padding: 216 products of 64 cycles a block against 100 of 64 and 100 of
// about 19).  Register r of lane l holds row 4 r + l / 16 of column l % 16, the
// 4x4x4 result row 16 + l / 16 (measured with one-hot operands).  The volume's
// K steps are axis-major (step ks: axis ks / NJ, nodes 4 (ks % NJ) + 0..3), so
// a lane reads the same nodes once for all axes; the lift's 4 Nfp flux rows
// are Nfp steps without padding.  Three barriers: the neighbour traces of all
// faces are requested ahead of the volume product, their fluxes formed at once.
//
// P2 takes its operands from registers (15 loads per wave).  P3's 25 steps need
// 100 registers and 50 loads per wave, which alone cost 10 us of a 60 us
// 48000-tet launch; a workgroup therefore keeps the table in LDS (16 KB; three
// workgroups per compute unit as the registers allow) and runs several blocks.
// Requesting the next block ahead gained nothing (50.9 against 50.1 us).  P3
// requests the update's operands ahead of the flux (60 us against 69 behind it).
//
// us per launch, before (the best of eight forms with one to four waves, a
// barrier pair per face and P3's rows padded to 32) and now: P2 3072 tets 7.9 /
// 6.0, 10368 11.9 / 9.6, 24576 20.5 / 15.3, 82944 49.4 / 38.5; P3 3072 12.5 / 9.2,
// 10368 23.0 / 17.3, 48000 67.1 / 50.5, 82944 118.5 / 95.  What bounds it: the
// larger launches move 3.9-4.6 TB/s of traffic (a copy: 5.1), the small ones are
// one block's chain (7 us for P3, of which the products are 0.9).
template <int Q> struct TileDim {
    static constexpr int NP = Dim<Q>::NP, NFP = Dim<Q>::NFP;
    static constexpr int NJ = (NP + 3) / 4, KSV = 3 * NJ, NST = KSV + NFP;  // K steps: per axis, volume, all
    static constexpr bool TAIL = NP > 16;                                   // rows 16 .. 19
    static constexpr int RS = NP + 1;                                       // staged row stride
    static constexpr int FS = 65;  // flux row stride: the face nodes of one column fall in different banks
    static constexpr int RF = (EPW * 4 * NFP + 255) / 256;                  // flux nodes per thread
    static constexpr int NTAB = NST * (TAIL ? 80 : 64);
    static constexpr bool LOOP = Q == 3;  // a workgroup runs several blocks
    // waves per SIMD that the registers allow, so workgroups per compute unit
    static constexpr int occ(bool ltsm) { return Q == 3 ? (ltsm ? 2 : 3) : ltsm ? 4 : 5; }
};
// A operands [step][lane] of rows 0 .. 15 (lane l: row l % 16, K row l / 16),
// behind them [step][16] of rows 16 .. 19 (entry 4 k + i).
__device__ double gTile[TileDim<2>::NTAB + TileDim<3>::NTAB];

typedef double f64x4 __attribute__((ext_vector_type(4)));
template <int Q, int FIRST, int N> struct TileMats {  // steps FIRST .. FIRST + N - 1 in registers
    using TD = TileDim<Q>;
    double m[N], x[TD::TAIL ? N : 1];
    __device__ __forceinline__ void load(int lane) {
        const double* t = gTile + (Q == 2 ? 0 : TileDim<2>::NTAB);
#pragma unroll
        for (int i = 0; i < N; ++i) m[i] = t[(FIRST + i) * 64 + lane];
        if constexpr (TD::TAIL) {
            const double* u = t + TD::NST * 64 + (lane >> 4) * 4 + (lane & 3);
#pragma unroll
            for (int i = 0; i < N; ++i) x[i] = u[(FIRST + i) * 16];
        }
    }
    __device__ __forceinline__ double rows(int i) const { return m[i]; }
    __device__ __forceinline__ double tail(int i) const { return x[i]; }
};
template <int Q> using TileVolume = TileMats<Q, 0, TileDim<Q>::KSV>;
template <int Q> using TileLift = TileMats<Q, TileDim<Q>::KSV, TileDim<Q>::NFP>;
template <int Q, int FIRST> struct TileTable {  // the same from a copy of the table in LDS
    const double *m, *x;
    __device__ __forceinline__ TileTable(const double* t, int lane)
        : m(t + FIRST * 64 + lane), x(t + TileDim<Q>::NST * 64 + FIRST * 16 + (lane >> 4) * 4 + (lane & 3)) {}
    __device__ __forceinline__ double rows(int i) const { return m[i * 64]; }
    __device__ __forceinline__ double tail(int i) const { return x[i * 16]; }
};

template <int Q> struct TileAcc {
    f64x4 a = {0., 0., 0., 0.};
    double x = 0.;
    template <typename M> __device__ __forceinline__ void step(const M& mat, int i, double b) {
        a = __builtin_amdgcn_mfma_f64_16x16x4f64(mat.rows(i), b, a, 0, 0, 0);
        if constexpr (TileDim<Q>::TAIL) x = __builtin_amdgcn_mfma_f64_4x4x4f64(mat.tail(i), b, x, 0, 0, 0);
    }
    // rows of the lane's column: f(row, value)
    template <typename F> __device__ __forceinline__ void rows(int q4, F f) const {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * r + q4 < TileDim<Q>::NP) f(4 * r + q4, a[r]);
        if constexpr (TileDim<Q>::TAIL) f(16 + q4, x);
    }
};

// curl at all nodes of the lane's column n from the staged rows: B[(a, j)][n] =
// sgn (g_a[m1] V_m2(j) - g_a[m2] V_m1(j)); padded columns take element 0 (their
// results are never stored)
template <int Q, typename M>
__device__ __forceinline__ void tile_volume(const double* S, const double* sG, int n, int q4, int ne, const M& mat,
                                            TileAcc<Q>& acc) {
    using TD = TileDim<Q>;
    constexpr int NJ = TD::NJ, NP = TD::NP;
    const int e = n < 6 * ne ? n / 6 : 0;
    const int s = n - 6 * (n / 6);
    const int m = s < 3 ? s : s - 3;
    const int m1 = m == 2 ? 0 : m + 1, m2 = m == 0 ? 2 : m - 1;  // (m+1)%3, (m+2)%3
    const int vb = e * 6 + (s < 3 ? 3 : 0);
    const double sgn = s < 3 ? -1. : 1.;
    const double* gE = sG + e * kGeo;
    double g1[3], g2[3], r1[NJ], r2[NJ];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        g1[ax] = sgn * gE[3 * ax + m1];
        g2[ax] = sgn * gE[3 * ax + m2];
    }
    const double* v1 = S + (vb + m1) * TD::RS;
    const double* v2 = S + (vb + m2) * TD::RS;
#pragma unroll
    for (int t = 0; t < NJ; ++t) {
        const int j = q4 + 4 * t;
        const bool in = NP % 4 == 0 || j < NP;  // j >= Np: zero operands
        r1[t] = in ? v1[in ? j : 0] : 0.;
        r2[t] = in ? v2[in ? j : 0] : 0.;
    }
#pragma unroll
    for (int ax = 0; ax < 3; ++ax)
#pragma unroll
        for (int t = 0; t < NJ; ++t) acc.step(mat, ax * NJ + t, fma(g1[ax], r2[t], -g2[ax] * r1[t]));
}

// + LIFT (the column's fluxes); F = the flux tile [f Nfp + k][FS]
template <int Q, typename M>
__device__ __forceinline__ void tile_lift(const double* F, int n, int q4, const M& mat, TileAcc<Q>& acc) {
#pragma unroll
    for (int i = 0; i < TileDim<Q>::NFP; ++i) acc.step(mat, i, F[(4 * i + q4) * TileDim<Q>::FS + n]);
}

template <int Q> struct TileShared {
    using TD = TileDim<Q>;
    double sY[EPW * 6 * TD::RS];
    double sF[4 * TD::NFP * TD::FS];
    double sG[EPW * kGeo];
    double sM[TD::LOOP ? TD::NTAB : 1];
    uint8_t sT[4 * ft_words(Q)];
};

// The thread's share of a block: stage input, geometry and connectivity.
template <int Q> struct TileIn {
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    using TD = TileDim<Q>;
    static constexpr int NP = TD::NP, NTH = 256;
    static constexpr int NIT = (EPW * 6 * NP / 2 + NTH - 1) / NTH;
    static_assert(EPW * kGeo / 2 <= NTH && ft_words(Q) <= NTH, "one load per thread");
    f64x2 y[NIT], g;
    int code[TD::RF];
    uint32_t keep;
    __device__ __forceinline__ void request(const StageArgs& a, int64_t blk, int tid) {
        const int64_t e0 = blk * EPW;
        const int ne = (int)((a.K - e0) < EPW ? (a.K - e0) : EPW);
        const f64x2* Y = reinterpret_cast<const f64x2*>((const double*)a.Y + e0 * 6 * NP);
        const f64x2* geo = reinterpret_cast<const f64x2*>((const double*)a.geo + e0 * kGeo);
        const int* conn = a.conn + e0 * 4;
#pragma unroll
        for (int r = 0; r < TD::RF; ++r) {
            const int it = tid + NTH * r;
            code[r] = it < ne * 4 * TD::NFP ? conn[it / TD::NFP] : -3;
        }
#pragma unroll
        for (int t = 0; t < NIT; ++t)
            if (tid + NTH * t < ne * 6 * NP / 2) y[t] = Y[tid + NTH * t];
        if (tid < ne * kGeo / 2) g = geo[tid];
        keep = a.imask ? (a.imask[blk] ^ (a.imask_inv ? 0xffffffffu : 0u)) : 0xffffffffu;
    }
    __device__ __forceinline__ void put(TileShared<Q>& sh, int ne, int tid) const {
#pragma unroll
        for (int t = 0; t < NIT; ++t) {
            const int v = 2 * (tid + NTH * t);
            if (tid + NTH * t < ne * 6 * NP / 2) {
                const bool on = (keep >> (v / (6 * NP))) & 1u;
                sh.sY[v + v / NP] = on ? y[t][0] : 0.;
                sh.sY[v + 1 + v / NP] = on ? y[t][1] : 0.;
            }
        }
        if (tid < ne * kGeo / 2) reinterpret_cast<f64x2*>(sh.sG)[tid] = g;
    }
};

template <int Q, bool MH, bool LTSM, int STREAM, bool BATCH = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TileDim<Q>::occ(LTSM), 8)))
void k_stage_tile(StageArgs args, int64_t per) {
    using TD = TileDim<Q>;
    constexpr int NP = TD::NP, NFP = TD::NFP, RS = TD::RS, FS = TD::FS, NTH = 256, RF = TD::RF;
    constexpr bool LOOP = TD::LOOP;
    __shared__ __align__(16) TileShared<Q> sh;

    // the workgroup's blocks: index, index + step, .. of its XCD's range, of one
    // member: a batch's workgroups (BATCH) are dealt out to the members that take
    // the step.  A form of its own: in one, single launches took 0.4 % longer.  The
    // test of mtab, which batches always have, keeps the compiler's schedule of
    // the loop: without it they took 5 % longer.
    unsigned index = blockIdx.x >> 3, step = gridDim.x >> 3;
    StageArgs a;
    if constexpr (BATCH) {
        a = args;
        if (args.mtab) {
            const unsigned live = *args.nlive;
            if (live == 0) return;
            const unsigned m = index % live;
            step = (step - m + live - 1) / live;
            index /= live;
            member_offsets<double>(args, args.order[m], a);
        }
    } else if (!member_args<double>(args, a)) {
        return;  // uniform per workgroup
    }
    const int64_t nblk = a.blist ? a.nblist : (a.K + EPW - 1) / EPW;
    const int64_t lo = (blockIdx.x & 7) * per, hi = lo + per < nblk ? lo + per : nblk;
    const double* __restrict__ Y = (const double*)a.Y;
    int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    for (int64_t at = lo + index; at < hi; at += step) {
        // what depends on the thread alone is formed anew for every block: kept
        // across blocks it would take the registers of the loads in flight
        if constexpr (LOOP) asm volatile("" : "+v"(tid));
        const int lane = tid & 63, q4 = lane >> 4, n = 16 * wave + (lane & 15);
        const int64_t blk = a.blist ? a.blist[at] : at;  // with a list only the listed element blocks
        const int64_t e0 = blk * EPW;
        const int ne = (int)((a.K - e0) < EPW ? (a.K - e0) : EPW);
        const int64_t base = e0 * 6 * NP;
        const int nvv = ne * 6 * NP / 2;  // 16-byte groups of the block's rows

        // ---- every load that depends on no other; the tables with the first block
        const bool first = !LOOP || at < lo + step;
        constexpr int NM = LOOP ? (TD::NTAB + NTH - 1) / NTH : 1;
        uint32_t tw;
        double m[NM];
        if (first && tid < ft_words(Q)) tw = cFaceTab[ft_off(Q) + tid];
        TileIn<Q> in;
        in.request(a, blk, tid);
        TileVolume<Q> vol;
        if constexpr (!LOOP) vol.load(lane);
        if (LOOP && first) {
#pragma unroll
            for (int i = 0; i < NM; ++i)
                if (tid + NTH * i < TD::NTAB) m[i] = gTile[TileDim<2>::NTAB + tid + NTH * i];
        }
        if (!first) __syncthreads();  // the update has read the staged rows of the block before
        if (first && tid < ft_words(Q)) reinterpret_cast<uint32_t*>(sh.sT)[tid] = tw;
        in.put(sh, ne, tid);
        if (LOOP && first) {
#pragma unroll
            for (int i = 0; i < NM; ++i)
                if (tid + NTH * i < TD::NTAB) sh.sM[tid + NTH * i] = m[i];
        }
        __syncthreads();

        // ---- neighbour traces of the thread's face nodes, in flight during the
        // volume product (a neighbour in the block is read from LDS)
        double nv[RF][6];
        int own[RF], nbo[RF];
        bool off[RF];
        const auto masked = [&](int64_t nb) {  // the neighbour's values count as zero
            return a.imask && !(((a.imask[nb / EPW] >> (int)(nb % EPW)) & 1u) ^ (uint32_t)a.imask_inv);
        };
        const auto& code = in.code;
#pragma unroll
        for (int r = 0; r < RF; ++r) {
            const int it = tid + NTH * r, t = it / NFP, k = it - t * NFP;
            own[r] = (t >> 2) * 6 * RS + sh.sT[code[r] != -3 ? (t & 3) * NFP + k : 0];
            nbo[r] = -1;
            off[r] = false;
            if (code[r] >= 0) {
                const int nn = sh.sT[4 * NFP + (((code[r] >> 3) & 3) * 6 + (code[r] & 7)) * NFP + k];
                const int64_t nb = code[r] >> 5;
                if (nb >= e0 && nb < e0 + ne) {
                    nbo[r] = (int)(nb - e0) * 6 * RS + nn;
                } else if (!LTSM && masked(nb)) {
#pragma unroll
                    for (int cc = 0; cc < 6; ++cc) nv[r][cc] = 0.;
                } else {
                    if (LTSM) off[r] = masked(nb);  // the mask travels with the traces
                    const double* q = Y + nb * 6 * NP + nn;
#pragma unroll
                    for (int cc = 0; cc < 6; ++cc) nv[r][cc] = q[cc * NP];
                }
            }
        }

        TileAcc<Q> acc;
        TileLift<Q> lift;
        if constexpr (LOOP) {
            tile_volume<Q>(sh.sY, sh.sG, n, q4, ne, TileTable<Q, 0>(sh.sM, lane), acc);
        } else {
            tile_volume<Q>(sh.sY, sh.sG, n, q4, ne, vol, acc);
            lift.load(lane);  // in flight during the flux
        }
        MfmaUpdateIn<double, Q, NTH, LTSM, STREAM> upd;
        if constexpr (LOOP) upd.fetch(a, base, nvv, tid);  // in flight during flux and lift

        // ---- upwind flux of the thread's face nodes
#pragma unroll
        for (int r = 0; r < RF; ++r) {
            if (code[r] == -3) continue;
            const int it = tid + NTH * r, t = it / NFP, k = it - t * NFP;
            const double* om = &sh.sY[own[r]];
            double Em[3], Hm[3], Ep[3], Hp[3], fx[6];
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                Em[cc] = om[cc * RS];
                Hm[cc] = om[(3 + cc) * RS];
            }
            if (nbo[r] >= 0) {
                const double* np = &sh.sY[nbo[r]];
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    Ep[cc] = np[cc * RS];
                    Hp[cc] = np[(3 + cc) * RS];
                }
            } else {
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    // PEC ghost: E+ = -E-, H+ = H-; impedance ghost (homogeneous
                    // part): zero exterior state
                    Ep[cc] = code[r] >= 0 ? (LTSM && off[r] ? 0. : nv[r][cc]) : code[r] == -1 ? -Em[cc] : 0.;
                    Hp[cc] = code[r] >= 0 ? (LTSM && off[r] ? 0. : nv[r][3 + cc]) : code[r] == -1 ? Hm[cc] : 0.;
                }
            }
            upwind3(&sh.sG[(t >> 2) * kGeo + 9 + 7 * (t & 3)], Em, Hm, Ep, Hp, fx);
            double* o = &sh.sF[((t & 3) * NFP + k) * FS + (t >> 2) * 6];
#pragma unroll
            for (int cc = 0; cc < 6; ++cc) o[cc] = fx[cc];
        }
        __syncthreads();

        // ---- lift; scaled right-hand side in place of the stage input (only this
        // thread still reads these values)
        if constexpr (LOOP) {
            tile_lift<Q>(sh.sF, n, q4, TileTable<Q, TD::KSV>(sh.sM, lane), acc);
        } else {
            upd.fetch(a, base, nvv, tid);
            tile_lift<Q>(sh.sF, n, q4, lift, acc);
        }
        if (n < 6 * ne) {
            const int e = n / 6, s = n - 6 * e;
            const double inv = s < 3 ? sh.sG[e * kGeo + 37] : sh.sG[e * kGeo + 38];
            const double sig = s < 3 ? sh.sG[e * kGeo + 39] : 0.;
            acc.rows(q4, [&](int i, double v) {
                double* p = &sh.sY[n * RS + i];
                *p = fma(inv, v, -sig * *p);
            });
        }
        __syncthreads();
        stage_update<double, Q, NTH, MH, LTSM, STREAM>(args, a, upd, blk, base, nvv, tid, [&](int v, double (&kv)[2]) {
            kv[0] = sh.sY[v + v / NP];
            kv[1] = sh.sY[v + 1 + v / NP];
        });
        if constexpr (!LOOP) return;
    }
}

// ---------------------------------------------------------------------------
// FP32 stage kernel with one column per lane.
//
// A block of 10 elements has 60 columns (element, component); lane n of every
// wave owns column n, and wave w its nodes 4 w .. 4 w + 3 (P3: five waves, P2:
// three).  The products run on v_mfma_f32_4x4x1_16b_f32 with the
// matrix rows broadcast (mfma_cols.h): the B operand of a K step is the lane's
// own value, so
//   * the reference derivatives D_a y need the lane's own row only (16-byte LDS
//     reads), no operands are built, no matrix row is padded (20 rows = five
//     groups of four; the 16-row tiles of v_mfma_f32_16x16x4 spend 3/8 of
//     their rows on padding), and the matrices of a wave take 4 + 3 registers;
//   * curl terms are exchanged between the six lanes of an element, the lift
//     of all four faces reads the lane's 4 Nfp fluxes (16-byte LDS reads), and
//     the right-hand side ends up with the lane that owns it.
// Every global load that does not depend on another one (stage input, geometry,
// connectivity, matrices, update operands) is requested at the start (P3: the
// update operands behind the volume product, which leaves room for seven waves
// per SIMD: 30.7 us per 48000-tet launch against 32.5; P2: 110 us against 115 per
// 384000-tet launch the early way); the neighbour traces follow behind one
// barrier, with consecutive lanes on the nodes of a face, whose values share
// cache lines.  Three barriers in all.
//
// us per launch, before (the best form on 16x16x4 tiles with the wave's columns
// split over its lanes) and now: P2 3072 tets 6.2 / 5.1, 24576 12.0 / 10.3,
// 82944 28.2 / 24.2, 384000 117.7 / 110.4, 64 members of 10368 186.7 / 184; P3
// 3072 8.9 / 6.2, 10368 13.6 / 10.0, 48000 36.5 / 30.7, 82944 56.8 / 49.7.  What
// bounds it: memory for the large P2 launches (1.15 GB of traffic per GB of
// the implementation's bytes, 4.8-5 TB/s, a 1 GiB copy's rate being 5.1);
// at P3 a block's chain of dependent steps and the vector units together (418
// vector instructions a wave, a quarter of them on the matrix cores).
// LDS rows: stage input [column][RS], flux [column][FS], both conflict-free
// for 16-byte accesses of consecutive columns (RS / 4 and FS / 4 odd).
template <int Q> struct ColDim {
    static constexpr int NP = Dim<Q>::NP, NFP = Dim<Q>::NFP;
    static constexpr int W = (NP + 3) / 4, NTH = 64 * W;   // waves, threads
    static constexpr int RS = 4 * W;
    static constexpr int FS = 4 * NFP + (NFP % 2 ? 0 : 4);
    static constexpr int NV = (3 * NP + 15) / 16, NL = (4 * NFP + 15) / 16;  // operand registers: D, LIFT
    static constexpr int NTAB = W * (NV + NL) * 64;
    static constexpr int RF = (EPW * 4 * NFP + NTH - 1) / NTH;  // flux nodes per thread
};
__host__ __device__ constexpr int col_off(int q) {
    return q <= 2 ? 0 : ColDim<2>::NTAB;
}
constexpr int kColTotal = ColDim<2>::NTAB + ColDim<3>::NTAB;
// Broadcast operands [wave][D, LIFT registers][lane]: lane l of register v holds
// row 4 wave + l % 4 of K step 16 v + l / 4; D's K steps are (node j, axis a) =
// (step / 3, step % 3), LIFT's (face, face node).
__device__ float gCol[kColTotal];

template <int Q> struct ColMats {
    using CD = ColDim<Q>;
    float mV[CD::NV], mL[CD::NL];
    __device__ __forceinline__ void load(int wave, int lane) {
        const float* t = gCol + col_off(Q) + wave * (CD::NV + CD::NL) * 64 + lane;
#pragma unroll
        for (int v = 0; v < CD::NV; ++v) mV[v] = t[64 * v];
#pragma unroll
        for (int v = 0; v < CD::NL; ++v) mL[v] = t[64 * (CD::NV + v)];
    }
};

// A column's lane: its element, component, and the lanes and metric terms the
// curl exchange needs (k_stage's, see there).
struct ColLane {
    int el, c, row, lane_p, lane_m, kp, km;
    bool act;
    __device__ __forceinline__ void init(int lane, int ne) {
        el = lane / 6;
        c = lane - 6 * el;
        act = el < ne;
        el = act ? el : 0;
        row = el * 6 + c;
        const int c3 = c < 3 ? c : c - 3;
        kp = c3 == 0 ? 2 : c3 - 1;
        km = c3 == 2 ? 0 : c3 + 1;
        const int sb = el * 6 + (c < 3 ? 3 : 0);
        lane_p = sb + (c3 == 0 ? 2 : c3 - 1);
        lane_m = sb + (c3 == 2 ? 0 : c3 + 1);
    }
};

// curl of the lane's column at the wave's nodes (E rows: -curl H, H rows: +curl
// E), from the staged rows; geo = the element's geometry.
template <int Q>
__device__ __forceinline__ f32x4 col_volume(const float* srow, const float* geo, const ColLane& L,
                                            const ColMats<Q>& mat) {
    using CD = ColDim<Q>;
    float y[CD::RS];
#pragma unroll
    for (int v = 0; v < CD::RS / 4; ++v) {
        const f32x4 t = reinterpret_cast<const f32x4*>(srow)[v];
#pragma unroll
        for (int u = 0; u < 4; ++u) y[4 * v + u] = t[u];
    }
    f32x4 d[3] = {};
    mfma_rows<CD::NP, 3>(mat.mV, y, d);
    const float sgn = L.c < 3 ? -1.f : 1.f;
    f32x4 pv = {0.f, 0.f, 0.f, 0.f}, mv = {0.f, 0.f, 0.f, 0.f}, acc;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const float gp = geo[3 * ax + L.kp], gm = geo[3 * ax + L.km];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            pv[u] = fmaf(gp, d[ax][u], pv[u]);
            mv[u] = fmaf(-gm, d[ax][u], mv[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] = sgn * (__shfl(pv[u], L.lane_p) + __shfl(mv[u], L.lane_m));
    return acc;
}

// acc + LIFT (the column's fluxes), faces 0, 1 on top of acc and faces 2, 3 in
// a sum of their own (two chains of dependent products instead of one).
template <int Q>
__device__ __forceinline__ f32x4 col_lift(const float* frow, const ColMats<Q>& mat, f32x4 acc) {
    using CD = ColDim<Q>;
    constexpr int NF4 = 4 * CD::NFP;
    float x[NF4];
#pragma unroll
    for (int v = 0; v < NF4 / 4; ++v) {
        const f32x4 t = reinterpret_cast<const f32x4*>(frow)[v];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[4 * v + u] = t[u];
    }
    f32x4 b = {0.f, 0.f, 0.f, 0.f};
    mfma_pair<NF4>(mat.mL, x, acc, b);
    return acc + b;
}

// Four consecutive values v .. v + 3 of the block's contiguous rows in LDS rows
// padded to RS (P2: 10 values in 12; pairs never straddle a row).
template <int Q> __device__ __forceinline__ void col_put(float* S, int v, f32x4 x) {
    if constexpr (ColDim<Q>::RS == ColDim<Q>::NP) {
        *reinterpret_cast<f32x4*>(S + v) = x;
    } else {
        constexpr int NP = ColDim<Q>::NP, PAD = ColDim<Q>::RS - NP;
        *reinterpret_cast<float2*>(S + v + v / NP * PAD) = make_float2(x[0], x[1]);
        *reinterpret_cast<float2*>(S + v + 2 + (v + 2) / NP * PAD) = make_float2(x[2], x[3]);
    }
}
template <int Q> __device__ __forceinline__ f32x4 col_get(const float* S, int v) {
    if constexpr (ColDim<Q>::RS == ColDim<Q>::NP) {
        return *reinterpret_cast<const f32x4*>(S + v);
    } else {
        constexpr int NP = ColDim<Q>::NP, PAD = ColDim<Q>::RS - NP;
        const float2 p = *reinterpret_cast<const float2*>(S + v + v / NP * PAD);
        const float2 q = *reinterpret_cast<const float2*>(S + v + 2 + (v + 2) / NP * PAD);
        return f32x4{p.x, p.y, q.x, q.y};
    }
}

template <int Q> struct ColShared {
    using CD = ColDim<Q>;
    float sY[EPW * 6 * CD::RS];
    float sF[EPW * 6 * CD::FS];
    float sG[EPW * kGeo];
    uint8_t sT[4 * ft_words(Q)];
};

template <int Q, bool MH, bool LTSM, int STREAM>
__global__ __launch_bounds__(ColDim<Q>::NTH) __attribute__((amdgpu_waves_per_eu(LTSM ? 5 : Q == 3 ? 7 : 5, 8)))
void k_stage_col(StageArgs args, int64_t per) {
    using CD = ColDim<Q>;
    constexpr int NP = CD::NP, NFP = CD::NFP, RS = CD::RS, FS = CD::FS, NTH = CD::NTH, RF = CD::RF;
    __shared__ __align__(16) ColShared<Q> sh;

    StageArgs a;
    if (!member_args<float>(args, a)) return;  // uniform per workgroup
    int64_t blk = xcd_block(per);
    if (a.blist) {  // only the listed element blocks
        if (blk >= a.nblist) return;
        blk = a.blist[blk];
    }
    const int64_t e0 = blk * EPW;
    if (e0 >= a.K) return;  // uniform per workgroup
    const float* __restrict__ Y = (const float*)a.Y;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ne = (int)((a.K - e0) < EPW ? (a.K - e0) : EPW);
    const int64_t base = e0 * 6 * NP;
    const int nvv = ne * 6 * NP / 4;  // 16-byte groups of the block's rows
    const uint32_t keep = a.imask ? (a.imask[blk] ^ (a.imask_inv ? 0xffffffffu : 0u)) : 0xffffffffu;

    // ---- every load that depends on no other
    constexpr int NIT = (EPW * 6 * NP / 4 + NTH - 1) / NTH, NG = (EPW * kGeo / 4 + NTH - 1) / NTH;
    constexpr int NT = (ft_words(Q) + NTH - 1) / NTH;
    int code[RF];
    f32x4 yin[NIT], gin[NG];
    uint32_t tw[NT];
    ColMats<Q> mat;
    MfmaUpdateIn<float, Q, NTH, LTSM, STREAM> upd;
#pragma unroll
    for (int r = 0; r < RF; ++r) {
        const int it = tid + NTH * r;
        code[r] = it < ne * 4 * NFP ? a.conn[e0 * 4 + it / NFP] : -3;
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
        if (tid + NTH * t < ft_words(Q)) tw[t] = cFaceTab[ft_off(Q) + tid + NTH * t];
#pragma unroll
    for (int t = 0; t < NIT; ++t)
        if (tid + NTH * t < nvv) yin[t] = reinterpret_cast<const f32x4*>(Y + base)[tid + NTH * t];
#pragma unroll
    for (int t = 0; t < NG; ++t)
        if (tid + NTH * t < ne * kGeo / 4)
            gin[t] = reinterpret_cast<const f32x4*>((const float*)a.geo + e0 * kGeo)[tid + NTH * t];
    mat.load(wave, lane);
    if constexpr (Q < 3) upd.fetch(a, base, nvv, tid);
#pragma unroll
    for (int t = 0; t < NT; ++t)
        if (tid + NTH * t < ft_words(Q)) reinterpret_cast<uint32_t*>(sh.sT)[tid + NTH * t] = tw[t];
#pragma unroll
    for (int t = 0; t < NIT; ++t) {
        const int v = 4 * (tid + NTH * t);
        if (tid + NTH * t < nvv) {
            if (!((keep >> (v / (6 * NP))) & 1u)) yin[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            col_put<Q>(sh.sY, v, yin[t]);
        }
    }
#pragma unroll
    for (int t = 0; t < NG; ++t)
        if (tid + NTH * t < ne * kGeo / 4) reinterpret_cast<f32x4*>(sh.sG)[tid + NTH * t] = gin[t];
    __syncthreads();

    // ---- neighbour traces of the thread's face nodes, in flight during the
    // volume product (a neighbour in the block is read from LDS)
    float nv[RF][6];
    int own[RF], nbo[RF];
    bool off[RF];
    const auto masked = [&](int64_t nb) {  // the neighbour's values count as zero
        return a.imask && !(((a.imask[nb / EPW] >> (int)(nb % EPW)) & 1u) ^ (uint32_t)a.imask_inv);
    };
#pragma unroll
    for (int r = 0; r < RF; ++r) {
        const int it = tid + NTH * r, t = it / NFP, k = it - t * NFP;
        own[r] = (t >> 2) * 6 * RS + sh.sT[code[r] != -3 ? (t & 3) * NFP + k : 0];
        nbo[r] = -1;
        off[r] = false;
        if (code[r] >= 0) {
            const int nn = sh.sT[4 * NFP + (((code[r] >> 3) & 3) * 6 + (code[r] & 7)) * NFP + k];
            const int64_t nb = code[r] >> 5;
            if (nb >= e0 && nb < e0 + ne) {
                nbo[r] = (int)(nb - e0) * 6 * RS + nn;
            } else if (!LTSM && masked(nb)) {
#pragma unroll
                for (int cc = 0; cc < 6; ++cc) nv[r][cc] = 0.f;
            } else {
                if (LTSM) off[r] = masked(nb);  // the mask travels with the traces
                const float* q = Y + nb * 6 * NP + nn;
#pragma unroll
                for (int cc = 0; cc < 6; ++cc) nv[r][cc] = q[cc * NP];
            }
        }
    }

    ColLane L;
    L.init(lane, ne);
    const float* gl = &sh.sG[L.el * kGeo];
    f32x4 acc = col_volume<Q>(&sh.sY[L.row * RS], gl, L, mat);
    if constexpr (Q == 3) upd.fetch(a, base, nvv, tid);  // in flight during flux and lift

    // ---- upwind flux of the thread's face nodes
#pragma unroll
    for (int r = 0; r < RF; ++r) {
        if (code[r] == -3) continue;
        const int it = tid + NTH * r, t = it / NFP, k = it - t * NFP;
        const float* om = &sh.sY[own[r]];
        float Em[3], Hm[3], Ep[3], Hp[3], fx[6];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            Em[cc] = om[cc * RS];
            Hm[cc] = om[(3 + cc) * RS];
        }
        if (nbo[r] >= 0) {
            const float* np = &sh.sY[nbo[r]];
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                Ep[cc] = np[cc * RS];
                Hp[cc] = np[(3 + cc) * RS];
            }
        } else {
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                // PEC ghost: E+ = -E-, H+ = H-; impedance ghost (homogeneous
                // part): zero exterior state
                Ep[cc] = code[r] >= 0 ? (LTSM && off[r] ? 0.f : nv[r][cc]) : code[r] == -1 ? -Em[cc] : 0.f;
                Hp[cc] = code[r] >= 0 ? (LTSM && off[r] ? 0.f : nv[r][3 + cc]) : code[r] == -1 ? Hm[cc] : 0.f;
            }
        }
        upwind3(&sh.sG[(t >> 2) * kGeo + 9 + 7 * (t & 3)], Em, Hm, Ep, Hp, fx);
        float* o = &sh.sF[(t >> 2) * 6 * FS + (t & 3) * NFP + k];
#pragma unroll
        for (int cc = 0; cc < 6; ++cc) o[cc * FS] = fx[cc];
    }
    __syncthreads();

    // ---- lift; scaled right-hand side in place of the stage input (only this
    // thread still reads these values)
    acc = col_lift<Q>(&sh.sF[L.row * FS], mat, acc);
    if (L.act) {
        const float inv = L.c < 3 ? gl[37] : gl[38];
        const float sig = L.c < 3 ? gl[39] : 0.f;
        f32x4* p = reinterpret_cast<f32x4*>(&sh.sY[L.row * RS + 4 * wave]);
        const f32x4 y = *p;
        f32x4 kv;
#pragma unroll
        for (int u = 0; u < 4; ++u) kv[u] = fmaf(inv, acc[u], -sig * y[u]);
        *p = kv;
    }
    __syncthreads();
    stage_update<float, Q, NTH, MH, LTSM, STREAM>(args, a, upd, blk, base, nvv, tid, [&](int v, float (&kv)[4]) {
        const f32x4 t = col_get<Q>(sh.sY, v);
#pragma unroll
        for (int u = 0; u < 4; ++u) kv[u] = t[u];
    });
}

// ---------------------------------------------------------------------------
// A whole period in one launch (PeriodArgs in launch.h), for meshes whose
// element blocks all fit on the device at once: a workgroup keeps a block of 10
// elements resident -- state, stage combination and low parts in registers,
// stage input and geometry in LDS, matrix fragments in registers -- and the
// stages run in a loop.  The traces of faces between blocks go through
// mailboxes of (value, epoch) pairs (tagged.h; the 2-D kernels do the same):
// after its update a block writes its traces into its neighbours' mailboxes
// and polls its own until they carry the stage's epoch.  Two buffers alternate
// between epochs; a block overwrites a mailbox two stages later, after it has
// read that neighbour's next epoch, which the neighbour wrote after reading
// this one.
//
// The faces of a period kernel's block: which traces leave it, which arrive,
// and the flux nodes of its threads.  LDS array S: the staged block [row][RS],
// behind it (offset XO) the received traces [face][component][face node],
// behind these (FO) the flux.
template <typename T, int Q, int NTH, int RS> struct PeriodFaces {
    static constexpr int NFP = Dim<Q>::NFP;
    static constexpr int NFACE = EPW * 4;
    static constexpr int XO = EPW * 6 * RS;
    static constexpr int CF = 6 * NFP;         // values of a mailbox
    static constexpr int RF = (NFACE * NFP + NTH - 1) / NTH;  // flux nodes per thread
    static constexpr int FO = XO + NFACE * CF;
    // mailbox values a thread keeps track of (20 of a block's 40 faces leaving
    // it; more, on meshes numbered worse, are looked up each time)
    static constexpr int RQ = (20 * CF + NTH - 1) / NTH;
    using X = Tagged<T>;
    struct Shared {
        int box[NFACE];        // mailbox j: the neighbour's mailbox ...
        uint8_t face[NFACE];   // ... and its local face 4 e + f
        uint8_t node[4 * NFP]; // own face nodes [f][k]
        int stop;
    };
    uint32_t trace[RF], place[RF];
    uint32_t mlds[RQ], mdst[RQ];
    int n;  // values of the block's mailboxes

    static __device__ __forceinline__ int table(int i) {
        return (int)((cFaceTab[ft_off(Q) + i / 4] >> (8 * (i % 4))) & 255u);
    }
    __device__ __forceinline__ void mail(const Shared& sh, int i, int& src, uint32_t& dst, int& rcv) const {
        const int j = i / CF, r = i - j * CF;
        const int cc = r / NFP, k = r - cc * NFP;
        const int t = sh.face[j];
        src = ((t >> 2) * 6 + cc) * RS + sh.node[(t & 3) * NFP + k];
        dst = (uint32_t)(sh.box[j] * CF + r) * X::W;
        rcv = XO + t * CF + r;
    }
    // first part: the shared tables (a barrier follows)
    __device__ __forceinline__ void tables(Shared& sh, const PeriodArgs& a, int64_t blk, int ne, int tid) {
        const int64_t e0 = blk * EPW;
        const int x0 = a.xstart[blk];
        n = (a.xstart[blk + 1] - x0) * CF;
        if (tid == 0) sh.stop = 0;
        if (tid < 4 * NFP) sh.node[tid] = (uint8_t)table(tid);
        if (tid < ne * 4) {
            const int id = a.xslot[e0 * 4 + tid], cd = a.conn[e0 * 4 + tid];
            if (id >= 0) {
                sh.face[id - x0] = (uint8_t)tid;
                sh.box[id - x0] = a.xslot[(int64_t)(cd >> 5) * 4 + ((cd >> 3) & 3)];
            }
        }
    }
    // second part: this thread's flux nodes and mailbox values.  trace: LDS
    // offsets of the own and the neighbour's first component; place: the face's
    // geometry (10 bits), the flux's place behind FO (14 bits: fo(f, k, e)) and
    // what the neighbour is (8 bits): the offset between its components, 0 on a
    // wall with the PEC ghost, 1 with the impedance ghost
    template <typename F>
    __device__ __forceinline__ void init(const Shared& sh, const PeriodArgs& a, int64_t e0, int ne, int tid, F fo) {
        static_assert(NFP > 1 && RS > 1 && RS < 256 && XO + NFACE * CF < 65536 && EPW * kGeo < 1024, "packed offsets");
#pragma unroll
        for (int r = 0; r < RF; ++r) {
            const int it = tid + NTH * r;
            const int t = it < NFACE * NFP ? it / NFP : 0, k = it < NFACE * NFP ? it % NFP : 0;
            const int e = t >> 2, f = t & 3;
            const int code = t < ne * 4 ? a.conn[e0 * 4 + t] : -2;
            const int own = e * 6 * RS + table(f * NFP + k);
            int nbo = own, what = code == -1 ? 0 : 1;
            if (code >= 0) {
                const int64_t nb = code >> 5;
                const int nf = (code >> 3) & 3;
                const int nn = table(4 * NFP + (nf * 6 + (code & 7)) * NFP + k);
                if (nb >= e0 && nb < e0 + ne) {
                    nbo = (int)(nb - e0) * 6 * RS + nn;
                    what = RS;
                } else {  // the neighbour's mailbox order: its own face nodes
                    int m = 0;
                    for (int q = 0; q < NFP; ++q)
                        if (table(nf * NFP + q) == nn) m = q;
                    nbo = XO + t * CF + m;
                    what = NFP;
                }
            }
            trace[r] = (uint32_t)own | ((uint32_t)nbo << 16);
            place[r] = (uint32_t)(e * kGeo + 9 + 7 * f) | ((uint32_t)fo(f, k, e) << 10) | ((uint32_t)what << 24);
        }
#pragma unroll
        for (int r = 0; r < RQ; ++r) {
            mlds[r] = mdst[r] = 0;
            if (tid + NTH * r < n) {
                int src, rcv;
                mail(sh, tid + NTH * r, src, mdst[r], rcv);
                mlds[r] = (uint32_t)src | ((uint32_t)rcv << 16);
            }
        }
    }
    // packed words stay packed: unpacked ahead of the loop they would take
    // three times the registers
    __device__ __forceinline__ void hold() {
#pragma unroll
        for (int r = 0; r < RF; ++r) asm volatile("" : "+v"(trace[r]), "+v"(place[r]));
#pragma unroll
        for (int r = 0; r < RQ; ++r) asm volatile("" : "+v"(mlds[r]), "+v"(mdst[r]));
    }
    // the block's traces into the neighbours' mailboxes (out: this epoch's buffer)
    __device__ __forceinline__ void publish(const Shared& sh, const T* S, unsigned long long* out, uint32_t epoch,
                                            int tid) const {
#pragma unroll
        for (int r = 0; r < RQ; ++r)
            if (tid + NTH * r < n) X::put(out + mdst[r], S[mlds[r] & 0xffffu], epoch);
        for (int i = tid + NTH * RQ; i < n; i += NTH) {
            int src, rcv;
            uint32_t dst;
            mail(sh, i, src, dst, rcv);
            X::put(out + dst, S[src], epoch);
        }
    }
    // waits for the block's own mailboxes (in: this epoch's buffer)
    __device__ __forceinline__ void receive(Shared& sh, T* S, Inbox<T, RQ, NTH>& box, const unsigned long long* in,
                                            uint32_t epoch, const PeriodArgs& a, int tid) const {
        const auto take = [&](int i, int r, T v) {
            int src, rcv = (int)(mlds[r < RQ ? r : 0] >> 16);
            uint32_t dst;
            if (r >= RQ) mail(sh, i, src, dst, rcv);
            S[rcv] = v;
        };
        bool ok;
        if constexpr (Q == 1) {
            // values beyond the tracked ones are requested before those are waited
            // for (randomly numbered 1296 tets FP64: 3.7 -> 3.2 us a stage; cube
            // order, where there are none, 2.8 -> 2.7.  P2 and P3, which track
            // more: 4.2 -> 4.9 and 5.2 -> 5.8 us)
            constexpr int RX = (8 * CF + NTH - 1) / NTH;
            Inbox<T, RX, NTH> more;
            if (n > NTH * RQ) more.request(in, NTH * RQ, n, tid);
            ok = box.settle_batch(in, 0, n, tid, epoch, a, take);
            for (int first = NTH * RQ; ok && first < n; first += NTH * RX) {
                if (first > NTH * RQ) more.request(in, first, n, tid);
                ok = more.settle_batch(in, first, n, tid, epoch, a, [&](int i, int, T v) { take(i, RQ, v); });
            }
        } else {
            ok = box.settle(in, n, tid, epoch, a, take);
        }
        if (!ok) sh.stop = 1;
    }
    // flux of every face node of the block (a barrier follows); geo = the
    // block's geometry
    __device__ __forceinline__ void flux(T* S, const T* geo, int cstride, int tid) const {
#pragma unroll
        for (int r = 0; r < RF; ++r) {
            if (tid + NTH * r >= NFACE * NFP) break;
            const T* om = &S[trace[r] & 0xffffu];
            const T* np = &S[trace[r] >> 16];
            const int what = place[r] >> 24;
            const int st = what > 1 ? what : RS;
            T Em[3], Hm[3], Ep[3], Hp[3], fx[6];
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                Em[cc] = om[cc * RS];
                Hm[cc] = om[(3 + cc) * RS];
                Ep[cc] = np[cc * st];
                Hp[cc] = np[(3 + cc) * st];
                if (what == 0) Ep[cc] = -Em[cc];          // PEC ghost: E+ = -E-, H+ = H-
                if (what == 1) Ep[cc] = Hp[cc] = T(0);    // impedance ghost (homogeneous part): zero exterior state
            }
            upwind3(&geo[place[r] & 1023u], Em, Hm, Ep, Hp, fx);
            T* o = &S[FO + ((place[r] >> 10) & 16383u)];
#pragma unroll
            for (int cc = 0; cc < 6; ++cc) o[cc * cstride] = fx[cc];
        }
    }
};

// Member, block and sizes of a period kernel's workgroup; false when it has
// nothing to do.
__device__ __forceinline__ bool period_block(const PeriodArgs& a, int64_t per, int& mem, int64_t& blk) {
    mem = a.order ? a.order[a.first + blockIdx.y] : 0;
    blk = xcd_block(per);
    return blk * EPW < a.K;
}

// FP64 P2 and P3, with the arithmetic of k_stage_tile: results agree with the
// stage launches bit for bit.
template <int Q, int OCC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(OCC, 8)))
void k_period_tile(PeriodArgs a, int64_t per) {
    using T = double;
    using TD = TileDim<Q>;
    constexpr int NP = TD::NP, NTH = 256, RS = TD::RS, FS = TD::FS;
    using PF = PeriodFaces<T, Q, NTH, RS>;
    constexpr int FO = PF::FO, NSH = FO + 4 * TD::NFP * FS;
    constexpr int PV = 16 / (int)sizeof(T);         // values of an update group
    constexpr int NIT = (EPW * 6 * NP / PV + NTH - 1) / NTH;
    typedef T V __attribute__((ext_vector_type(PV)));
    __shared__ __align__(16) T S[NSH];
    __shared__ T sG[EPW * kGeo];
    __shared__ typename PF::Shared sh;

    int mem;
    int64_t blk;
    if (!period_block(a, per, mem, blk)) return;  // uniform per workgroup
    const int64_t e0 = blk * EPW;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int q4 = lane >> 4, n = 16 * wave + (lane & 15), upd = tid;
    const int ne = (int)((a.K - e0) < EPW ? (a.K - e0) : EPW);
    const int nvv = ne * 6 * NP / PV;
    const int64_t base = (int64_t)mem * a.bstride + e0 * 6 * NP;
    const int M = a.msteps ? a.msteps[mem] : a.M;
    const int NS = a.scheme == 2 ? 2 : 4;

    TileVolume<Q> vol;
    TileLift<Q> lift;
    vol.load(lane);
    lift.load(lane);
    // state: 16-byte groups v = tid + NTH t of the block's rows
    V up[NIT], ap[NIT];
    const T* geo = (const T*)a.geo + (int64_t)mem * a.gstride + e0 * kGeo;
    for (int i = tid; i < ne * kGeo; i += NTH) sG[i] = geo[i];
    for (int i = tid; i < NSH; i += NTH) S[i] = T(0);
    PF pf;
    pf.tables(sh, a, blk, ne, tid);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NIT; ++t) {
        const int vv = tid + NTH * t;
        up[t] = V(T(0));
        ap[t] = V(T(0));
        if (vv < nvv) {
            up[t] = *reinterpret_cast<const V*>((const T*)a.U + base + PV * vv);
            const int v = PV * vv;
#pragma unroll
            for (int u = 0; u < PV; ++u) S[v + u + (v + u) / NP] = up[t][u];
        }
    }
    pf.init(sh, a, e0, ne, tid, [](int f, int k, int e) { return (f * TD::NFP + k) * FS + e * 6; });

    uint32_t epoch = a.epoch;
    const int64_t half = (int64_t)a.members * a.next * (PF::CF * PF::X::W);  // words of one buffer
    unsigned long long* const xch = a.xch + (int64_t)mem * a.next * (PF::CF * PF::X::W);
    const unsigned long long* const inbox = xch + (int64_t)a.xstart[blk] * (PF::CF * PF::X::W);
    const uint32_t sm = a.src_rows > 0 ? (a.smask ? a.smask[(int64_t)mem * ((a.K + EPW - 1) / EPW) + blk] : 0xffffffffu) : 0u;
    // RK4 with the filter ends with one more right-hand side at the last level
    const bool tail = a.filter && NS == 4;
    __syncthreads();
    pf.publish(sh, S, xch + (epoch & 1) * half, epoch, tid);
    for (int m = 0; m < M + (tail ? 1 : 0); ++m) {
        const int ns = m < M ? NS : 1;
        for (int s = 0; s < ns; ++s) {
            pf.hold();
            // indices are formed anew in every stage: ahead of the loop they and
            // the geometry behind them would take the registers
            asm volatile("" : "+v"(q4), "+v"(n), "+v"(upd));
            const double* tab = a.mtab + (((int64_t)(m < M ? m : a.M) * NS + s) * a.members + mem) * kMemberParams;
            const T cy = (T)tab[0], ca = (T)tab[1], cu = (T)tab[2], scos = (T)tab[3], ssin = (T)tab[4];
            // request the neighbours' traces; they travel during the volume product
            const unsigned long long* const in = inbox + (epoch & 1) * half;
            Inbox<T, PF::RQ, NTH> box;
            box.request(in, 0, pf.n, tid);

            TileAcc<Q> acc;
            tile_volume<Q>(S, sG, n, q4, ne, vol, acc);

            pf.receive(sh, S, box, in, epoch, a, tid);
            __syncthreads();
            if (sh.stop) return;
            pf.flux(S, sG, 1, tid);
            __syncthreads();

            // ---- lift; scaled right-hand side into the staged rows, in place
            tile_lift<Q>(S + FO, n, q4, lift, acc);
            if (n < 6 * ne) {
                const int e = n / 6, sc = n - 6 * e;
                const T inv = sc < 3 ? sG[e * kGeo + 37] : sG[e * kGeo + 38];
                const T sig = sc < 3 ? sG[e * kGeo + 39] : T(0);
                acc.rows(q4, [&](int i, T v) {
                    T* p = &S[n * RS + i];
                    *p = fma(inv, v, -sig * *p);
                });
            }
            __syncthreads();

            // ---- update of the thread's groups, next stage input into LDS
            const bool last = s == NS - 1;
#pragma unroll
            for (int t = 0; t < NIT; ++t) {
                const int vv = upd + NTH * t;
                if (vv >= nvv) continue;
                const int v = PV * vv;
                const int64_t gi = base + v;
                T kv[PV];
#pragma unroll
                for (int u = 0; u < PV; ++u) kv[u] = S[v + u + (v + u) / NP];
                if (sm) {
                    auto takes = [&](int row) { return row - 6 * (row / 6) < a.src_rows && ((sm >> (row / 6)) & 1u); };
                    if (takes(v / NP) || takes((v + PV - 1) / NP)) {
                        const int64_t si = (int64_t)mem * a.sstride + e0 * 6 * NP + v;
                        const V srv = *reinterpret_cast<const V*>((const T*)a.Sre + si);
                        const V siv = *reinterpret_cast<const V*>((const T*)a.Sim + si);
#pragma unroll
                        for (int u = 0; u < PV; ++u)
                            if (takes((v + u) / NP)) kv[u] = fma(scos, srv[u], fma(-ssin, siv[u], kv[u]));
                    }
                }
                if (a.filter && s == 0) {  // the stage input is the state
                    const double fa_re = tab[5], fa_im = tab[6], fb_re = tab[7], fb_im = tab[8];
#pragma unroll
                    for (int u = 0; u < PV; ++u) {
                        const double ud = (double)up[t][u], kd = (double)kv[u];
                        a.Fre[gi + u] = fma(fa_re, ud, fma(fb_re, kd, a.Fre[gi + u]));
                        a.Fim[gi + u] = fma(fa_im, ud, fma(fb_im, kd, a.Fim[gi + u]));
                    }
                }
                if (m >= M) continue;  // the last level's right-hand side: filter only
                V y;
                if (!last) {
#pragma unroll
                    for (int u = 0; u < PV; ++u) {
                        if (NS == 4)
                            ap[t][u] = s > 0 ? fma(ca, kv[u], ap[t][u]) : fma(ca, kv[u], up[t][u]);
                        y[u] = fma(cy, kv[u], up[t][u]);
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < PV; ++u) up[t][u] = fma(cu, kv[u], NS == 4 ? ap[t][u] : up[t][u]);
                    y = up[t];
                }
#pragma unroll
                for (int u = 0; u < PV; ++u) S[v + u + (v + u) / NP] = y[u];
            }
            if (m + 1 < M || (m < M && (!last || tail))) {
                ++epoch;
                __syncthreads();
                pf.publish(sh, S, xch + (epoch & 1) * half, epoch, tid);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < NIT; ++t) {
        const int vv = tid + NTH * t;
        if (vv >= nvv) continue;
        *reinterpret_cast<V*>((T*)a.U + base + PV * vv) = up[t];
    }
}

// FP32: one column per lane, the arithmetic of k_stage_col.  A thread owns
// nodes 4 wave .. 4 wave + 3 of its lane's column throughout -- state, stage
// combination, right-hand side -- so nothing is exchanged between the lift and
// the next stage input: three barriers a stage.  What bounds it: one exchange
// (0.4-0.6 us one way) and a block's chain per stage -- 3.5 us at P2 and 3072
// tets, 4.4 us at P3 -- and with several blocks on a compute unit their vector
// instructions (P2, 15300 tets: 6.4 us).  OCC: waves per SIMD, what the registers
// allow without spills (95 of 96 at P3).
template <int Q, int OCC>
__global__ __launch_bounds__(ColDim<Q>::NTH) __attribute__((amdgpu_waves_per_eu(OCC, 8)))
void k_period_col(PeriodArgs a, int64_t per) {
    using CD = ColDim<Q>;
    constexpr int NP = CD::NP, NFP = CD::NFP, RS = CD::RS, FS = CD::FS, NTH = CD::NTH;
    using PF = PeriodFaces<float, Q, NTH, RS>;
    constexpr int FO = PF::FO, NSH = FO + EPW * 6 * FS;
    __shared__ __align__(16) float S[NSH];
    __shared__ float sG[EPW * kGeo];
    __shared__ typename PF::Shared sh;

    int mem;
    int64_t blk;
    if (!period_block(a, per, mem, blk)) return;  // uniform per workgroup
    const int64_t e0 = blk * EPW;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ne = (int)((a.K - e0) < EPW ? (a.K - e0) : EPW);
    const int M = a.msteps ? a.msteps[mem] : a.M;
    const int NS = a.scheme == 2 ? 2 : 4;
    ColLane L;
    L.init(lane, ne);
    ColMats<Q> mat;
    mat.load(wave, lane);
    // uniform bases, 32-bit lane offsets
    const int64_t base = (int64_t)mem * a.bstride + e0 * 6 * NP, sbase = (int64_t)mem * a.sstride + e0 * 6 * NP;
    uint32_t at = (uint32_t)(L.row * NP + 4 * wave);
    float* const U = (float*)a.U + base;
    uint16_t* const Ulo = (uint16_t*)a.Ulo + base;
    const int nn = !L.act ? 0 : NP - 4 * wave < 4 ? NP - 4 * wave : 4;  // nodes of this thread
    const float* geo = (const float*)a.geo + (int64_t)mem * a.gstride + e0 * kGeo;
    for (int i = tid; i < ne * kGeo; i += NTH) sG[i] = geo[i];
    for (int i = tid; i < NSH; i += NTH) S[i] = 0.f;
    PF pf;
    pf.tables(sh, a, blk, ne, tid);
    __syncthreads();
    f32x4 up = {0.f, 0.f, 0.f, 0.f}, ap = up;
    uint32_t lop[2] = {0u, 0u};  // bfloat16 low parts
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (u < nn) {
            up[u] = U[at + u];
            lop[u / 2] |= (uint32_t)Ulo[at + u] << (16 * (u % 2));
        }
    f32x4* const own = reinterpret_cast<f32x4*>(&S[L.row * RS + 4 * wave]);
    if (L.act) *own = up;
    pf.init(sh, a, e0, ne, tid, [](int f, int k, int e) { return e * 6 * FS + f * NFP + k; });
    const bool src = L.act && L.c < a.src_rows &&
                     (!a.smask || ((a.smask[(int64_t)mem * ((a.K + EPW - 1) / EPW) + blk] >> L.el) & 1u));

    uint32_t epoch = a.epoch;
    const int64_t half = (int64_t)a.members * a.next * PF::CF;  // words of one buffer
    unsigned long long* const xch = a.xch + (int64_t)mem * a.next * PF::CF;
    const unsigned long long* const inbox = xch + (int64_t)a.xstart[blk] * PF::CF;
    // RK4 with the filter ends with one more right-hand side at the last level
    const bool tail = a.filter && NS == 4;
    __syncthreads();
    pf.publish(sh, S, xch + (epoch & 1) * half, epoch, tid);
    for (int m = 0; m < M + (tail ? 1 : 0); ++m) {
        const int ns = m < M ? NS : 1;
        for (int s = 0; s < ns; ++s) {
            pf.hold();
            asm volatile("" : "+v"(at));
            // an offset of zero that the compiler cannot see: geometry is read
            // from LDS in every stage (ahead of the loop it would take registers)
            int z = 0;
            asm volatile("" : "+v"(z));
            const double* tab = a.mtab + (((int64_t)(m < M ? m : a.M) * NS + s) * a.members + mem) * kMemberParams;
            const auto coef = [&](int k) {  // uniform: kept in scalar registers
                return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint((float)tab[k])));
            };
            const float cy = coef(0), ca = coef(1), cu = coef(2), scos = coef(3), ssin = coef(4);
            // request the neighbours' traces; they travel during the volume product
            const unsigned long long* const in = inbox + (epoch & 1) * half;
            Inbox<float, PF::RQ, NTH> box;
            box.request(in, 0, pf.n, tid);
            const float* gl = &sG[L.el * kGeo + z];
            f32x4 acc = col_volume<Q>(&S[L.row * RS], gl, L, mat);

            pf.receive(sh, S, box, in, epoch, a, tid);
            __syncthreads();
            if (sh.stop) return;
            pf.flux(S, sG + z, FS, tid);
            __syncthreads();
            acc = col_lift<Q>(&S[FO + L.row * FS], mat, acc);

            const float inv = L.c < 3 ? gl[37] : gl[38];
            const float sig = L.c < 3 ? gl[39] : 0.f;
            const f32x4 yo = *own;
            f32x4 kv;
#pragma unroll
            for (int u = 0; u < 4; ++u) kv[u] = fmaf(inv, acc[u], -sig * yo[u]);
            if (src) {
                const float* const Sre = (const float*)a.Sre + sbase;
                const float* const Sim = (const float*)a.Sim + sbase;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (u < nn)
                        kv[u] = fmaf(scos, Sre[at + u],
                                     fmaf(-ssin, Sim[at + u], kv[u]));
            }
            if (a.filter && s == 0) {
                const double fa_re = tab[5], fa_im = tab[6], fb_re = tab[7], fb_im = tab[8];
                double* const Fre = a.Fre + base;
                double* const Fim = a.Fim + base;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (u < nn) {
                        const double ud = (double)yo[u], kd = (double)kv[u];
                        Fre[at + u] = fma(fa_re, ud, fma(fb_re, kd, Fre[at + u]));
                        Fim[at + u] = fma(fa_im, ud, fma(fb_im, kd, Fim[at + u]));
                    }
            }
            if (m >= M) break;  // the last level's right-hand side: filter only
            const bool last = s == NS - 1;
            f32x4 yn;
            if (!last) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (NS == 4) ap[u] = s > 0 ? fmaf(ca, kv[u], ap[u]) : ca * kv[u];
                    yn[u] = fmaf(cy, kv[u], up[u]);
                }
            } else {
                float e[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float lo = from_bf16(u % 2 ? lop[u / 2] >> 16 : lop[u / 2] & 0xffffu);
                    float sum;
                    two_sum(up[u], NS == 4 ? fmaf(cu, kv[u], ap[u]) + lo : fmaf(cu, kv[u], lo), sum, e[u]);
                    up[u] = sum;
                }
                lop[0] = (uint32_t)to_bf16(e[0]) | ((uint32_t)to_bf16(e[1]) << 16);
                lop[1] = (uint32_t)to_bf16(e[2]) | ((uint32_t)to_bf16(e[3]) << 16);
                yn = up;
            }
            if (m + 1 < M || !last || tail) {
                ++epoch;
                if (L.act) *own = yn;  // every other reader of the old value is behind the flux's barrier
                __syncthreads();
                pf.publish(sh, S, xch + (epoch & 1) * half, epoch, tid);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (u < nn) {
            U[at + u] = up[u];
            Ulo[at + u] = (uint16_t)(u % 2 ? lop[u / 2] >> 16 : lop[u / 2] & 0xffffu);
        }
}

// P1 with the arithmetic of k_stage: lane = (element, component), each wave
// one of the four nodes of every row.
template <typename T>
__global__ __launch_bounds__(256) void k_period_p1(PeriodArgs a, int64_t per) {
    using PF = PeriodFaces<T, 1, 256, 5>;
    constexpr bool COMP = std::is_same<T, float>::value;
    constexpr int NP = 4, NFP = 3, NF4 = 4 * NFP, NTH = 256, RS = NP + 1, FO = PF::FO;
    constexpr int MO = mat_off(1), LO = MO + 3 * NP * NP;
    constexpr int NSH = FO + EPW * 6 * NF4;
    __shared__ T S[NSH];
    __shared__ T sG[EPW * kGeo];
    __shared__ typename PF::Shared sh;

    int mem;
    int64_t blk;
    if (!period_block(a, per, mem, blk)) return;  // uniform per workgroup
    const int64_t e0 = blk * EPW;
    const int tid = threadIdx.x, lane = tid & 63;
    const int i = __builtin_amdgcn_readfirstlane(tid >> 6);  // the wave's node
    const int ne = (int)((a.K - e0) < EPW ? (a.K - e0) : EPW);
    const int M = a.msteps ? a.msteps[mem] : a.M;
    const int NS = a.scheme == 2 ? 2 : 4;
    const int el = lane / 6, c = lane - 6 * el;
    const bool act = el < ne;
    const int elc = act ? el : 0;
    const int row = elc * 6 + c;
    const int64_t at = (int64_t)mem * a.bstride + (e0 * 6 + row) * NP + i;
    const T* geo = (const T*)a.geo + (int64_t)mem * a.gstride + e0 * kGeo;
    for (int k = tid; k < ne * kGeo; k += NTH) sG[k] = geo[k];
    for (int k = tid; k < NSH; k += NTH) S[k] = T(0);
    PF pf;
    pf.tables(sh, a, blk, ne, tid);
    __syncthreads();
    T up = act ? ((const T*)a.U)[at] : T(0), y = up, ap = T(0);
    float lo = 0.f;
    if constexpr (COMP)
        if (act) lo = from_bf16(((const uint16_t*)a.Ulo)[at]);
    if (act) S[row * RS + i] = y;
    pf.init(sh, a, e0, ne, tid, [](int f, int k, int e) { return e * 6 * NF4 + f * NFP + k; });
    // the node's matrix rows, the lane's metric terms
    T D[3][NP], L[NF4];
    const T* Mt = mats<T>();
#pragma unroll
    for (int ax = 0; ax < 3; ++ax)
#pragma unroll
        for (int j = 0; j < NP; ++j) D[ax][j] = Mt[MO + (ax * NP + i) * NP + j];
#pragma unroll
    for (int k = 0; k < NF4; ++k) L[k] = Mt[LO + i * NF4 + k];
    const int c3 = c < 3 ? c : c - 3;
    const int kp = c3 == 0 ? 2 : c3 - 1, km = c3 == 2 ? 0 : c3 + 1;
    const int sb = elc * 6 + (c < 3 ? 3 : 0);
    const int lane_p = sb + (c3 == 0 ? 2 : c3 - 1), lane_m = sb + (c3 == 2 ? 0 : c3 + 1);
    const T* gg = &sG[elc * kGeo];
    T gp[3], gm[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        gp[ax] = gg[3 * ax + kp];
        gm[ax] = gg[3 * ax + km];
    }
    const T inv = c < 3 ? gg[37] : gg[38];
    const T sig = c < 3 ? gg[39] : T(0);
    const T sgn = c < 3 ? T(-1) : T(1);
    const bool src = act && c < a.src_rows &&
                     (!a.smask || ((a.smask[(int64_t)mem * ((a.K + EPW - 1) / EPW) + blk] >> elc) & 1u));
    T sr = T(0), si = T(0);
    if (src) {
        const int64_t so = (int64_t)mem * a.sstride + (e0 * 6 + row) * NP + i;
        sr = ((const T*)a.Sre)[so];
        si = ((const T*)a.Sim)[so];
    }

    uint32_t epoch = a.epoch;
    const int64_t half = (int64_t)a.members * a.next * (PF::CF * PF::X::W);  // words of one buffer
    unsigned long long* const xch = a.xch + (int64_t)mem * a.next * (PF::CF * PF::X::W);
    const unsigned long long* const inbox = xch + (int64_t)a.xstart[blk] * (PF::CF * PF::X::W);
    const bool tail = a.filter && NS == 4;
    __syncthreads();
    pf.publish(sh, S, xch + (epoch & 1) * half, epoch, tid);
    for (int m = 0; m < M + (tail ? 1 : 0); ++m) {
        const int ns = m < M ? NS : 1;
        for (int s = 0; s < ns; ++s) {
            const double* tab = a.mtab + (((int64_t)(m < M ? m : a.M) * NS + s) * a.members + mem) * kMemberParams;
            const T cy = (T)tab[0], ca = (T)tab[1], cu = (T)tab[2], scos = (T)tab[3], ssin = (T)tab[4];
            const unsigned long long* const in = inbox + (epoch & 1) * half;
            Inbox<T, PF::RQ, NTH> box;
            box.request(in, 0, pf.n, tid);
            // ---- volume term of the node
            T yr[NP], pv = T(0), mv = T(0);
#pragma unroll
            for (int j = 0; j < NP; ++j) yr[j] = S[row * RS + j];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                T d = T(0);
#pragma unroll
                for (int j = 0; j < NP; ++j) d = fma(D[ax][j], yr[j], d);
                pv = fma(gp[ax], d, pv);
                mv = fma(-gm[ax], d, mv);
            }
            T acc = sgn * (__shfl(pv, lane_p) + __shfl(mv, lane_m));

            pf.receive(sh, S, box, in, epoch, a, tid);
            __syncthreads();
            if (sh.stop) return;
            pf.flux(S, sG, NF4, tid);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NF4; ++k) acc = fma(L[k], S[FO + row * NF4 + k], acc);

            T kv = fma(inv, acc, -sig * y);
            if (src) kv = fma(scos, sr, fma(-ssin, si, kv));
            if (a.filter && s == 0 && act) {
                const double ud = (double)y, kd = (double)kv;
                a.Fre[at] = fma(tab[5], ud, fma(tab[7], kd, a.Fre[at]));
                a.Fim[at] = fma(tab[6], ud, fma(tab[8], kd, a.Fim[at]));
            }
            if (m >= M) break;  // the last level's right-hand side: filter only
            const bool last = s == NS - 1;
            if (!last) {
                if (NS == 4) ap = s > 0 ? fma(ca, kv, ap) : COMP ? ca * kv : fma(ca, kv, y);
                y = fma(cy, kv, up);
            } else {
                if constexpr (COMP) {
                    float sum, e;
                    two_sum(up, NS == 4 ? fma(cu, kv, ap) + lo : fma(cu, kv, lo), sum, e);
                    up = sum;
                    lo = from_bf16(to_bf16(e));
                } else {
                    up = fma(cu, kv, NS == 4 ? ap : up);
                }
                y = up;
            }
            if (m + 1 < M || !last || tail) {
                ++epoch;
                if (act) S[row * RS + i] = y;  // read in this stage before the flux's barriers
                __syncthreads();
                pf.publish(sh, S, xch + (epoch & 1) * half, epoch, tid);
            }
        }
    }
    if (act) {
        ((T*)a.U)[at] = up;
        if constexpr (COMP) ((uint16_t*)a.Ulo)[at] = to_bf16(lo);
    }
}

// One 16x16x4 matrix-core product with the lane layout that k_stage_tile and
// k_period_tile assume in FP64 (a single 64-lane wave): lane l takes A[l % 16][l / 16] and
// B[l / 16][l % 16] and returns D[Mfma<T>::row(l / 16, r)][l % 16], r = 0..3.
template <typename T>
__global__ __launch_bounds__(64) void k_mfma_probe(const double* __restrict__ A, const double* __restrict__ B,
                                                   double* __restrict__ D) {
    const int l = threadIdx.x;
    const T a = (T)A[(l % 16) * 4 + l / 16];
    const T b = (T)B[(l / 16) * 16 + l % 16];
    typename Mfma<T>::acc_t c = {T(0), T(0), T(0), T(0)};
    c = Mfma<T>::mma(a, b, c);
#pragma unroll
    for (int r = 0; r < 4; ++r) D[Mfma<T>::row(l / 16, r) * 16 + l % 16] = (double)c[r];
}

template <typename T>
__global__ void k_to_field(const double* __restrict__ X, T* __restrict__ U, uint16_t* __restrict__ Ulo, int64_t n,
                           int Np, int flipH) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double x = X[i];
        if (flipH && ((i / Np) % 6) >= 3) x = -x;
        const T hi = (T)x;
        U[i] = hi;
        if constexpr (std::is_same<T, float>::value)
            if (Ulo) Ulo[i] = to_bf16((float)(x - (double)hi));
    }
}

template <typename T>
__global__ void k_from_field(const T* __restrict__ U, const uint16_t* __restrict__ Ulo, double* __restrict__ Yo,
                             const double* __restrict__ sub, int64_t n, int Np, int flipH) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double x = (double)U[i];
        if constexpr (std::is_same<T, float>::value)
            if (Ulo) x += (double)from_bf16(Ulo[i]);
        if (flipH && ((i / Np) % 6) >= 3) x = -x;
        if (sub) x -= sub[i];
        Yo[i] = x;
    }
}

template <typename T>
__global__ void k_copy(const T* __restrict__ s, T* __restrict__ d, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        d[i] = s[i];
}

__global__ void k_zero(uint32_t* p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// One 64-lane workgroup per element block: bit e of mask[block] is set when
// element e has a nonzero source value (either part, any row or harmonic).
template <typename T>
__global__ __launch_bounds__(64) void k_source_mask(const T* Sre, const T* Sim, int nharm, int64_t hstride,
                                                    int64_t K, int np6, uint32_t* mask) {
    const int64_t blk = blockIdx.x;
    const int64_t e0 = blk * EPW;
    const int ne = (int)((K - e0) < EPW ? (K - e0) : EPW);
    const int n = ne * np6;
    uint32_t bits = 0;
    for (int h = 0; h < nharm; ++h)
        for (int v = threadIdx.x; v < n; v += 64) {
            const int64_t g = h * hstride + e0 * np6 + v;
            if ((Sre && Sre[g] != T(0)) || (Sim && Sim[g] != T(0))) bits |= 1u << (v / np6);
        }
    for (int o = 32; o > 0; o >>= 1) bits |= (uint32_t)__shfl_xor((int)bits, o, 64);
    if (threadIdx.x == 0) mask[blk] = bits;
}

// ---- local time stepping: elementwise combinations of field vectors (field
// precision T, coefficients in FP64).  Row masks use the per-block element
// words of the stage kernels' masks (bit e of word b: element b EPW + e).
__device__ __forceinline__ bool lts_row_on(const uint32_t* mask, int inv, int64_t i, int np6) {
    const int64_t e = i / np6;
    return ((mask[e / EPW] >> (int)(e % EPW)) & 1u) ^ (uint32_t)inv;
}

// Values an elementwise LTS kernel visits: all n, or (blist non-null) the
// rows of the listed element blocks; returns the count and maps a visit
// index to the value index.
struct LtsRange {
    const int* blist;
    int64_t nb, n, per;  // per = EPW * 6 Np values of a block
    __device__ __forceinline__ int64_t count() const { return blist ? nb * per : n; }
    __device__ __forceinline__ int64_t at(int64_t f) const {
        if (!blist) return f;
        const int64_t b = f / per;
        return (int64_t)blist[b] * per + (f - b * per);
    }
};

// z = a y + b rows(x), rows(x) = x on the mask's rows (all rows when mask is
// null), 0 elsewhere; y nullable (= 0); z may alias y
template <typename T>
__global__ void k_lts_axpy(LtsRange rg, int np6, const uint32_t* mask, int inv, double a, const T* y, double b,
                           const T* x, T* z) {
    const int64_t cnt = rg.count();
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < cnt; v += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = rg.at(v);
        if (i >= rg.n) continue;
        const T xv = (!mask || lts_row_on(mask, inv, i, np6)) ? x[i] : T(0);
        z[i] = (y ? (T)a * y[i] : T(0)) + (T)b * xv;
    }
}

// Rows outside the mask (the coarse unknowns away from the fine region):
// z += sum_j al_j W_j + sc Sre - ss Sim (Sre nullable; source rows only where
// the source mask and the row's component allow)
template <typename T>
__global__ void k_lts_closed(int64_t n, int np6, int Np, const uint32_t* mask, const T* W0, const T* W1, const T* W2,
                             const T* W3, int nw, double a0, double a1, double a2, double a3, const T* Sre,
                             const T* Sim, int src_rows, double sc, double ss, T* z) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (lts_row_on(mask, 0, i, np6)) continue;
        T acc = z[i];
        if (nw > 0) acc += (T)a0 * W0[i];
        if (nw > 1) acc += (T)a1 * W1[i];
        if (nw > 2) acc += (T)a2 * W2[i];
        if (nw > 3) acc += (T)a3 * W3[i];
        if (Sre && ((i / Np) % 6) < src_rows) acc += (T)sc * Sre[i] - (T)ss * Sim[i];
        z[i] = acc;
    }
}

// Adjoint Taylor weights of the rows outside the mask (every coarse unknown):
// wb_j = al_j zbar there; the mask's rows keep what the substeps accumulated.
template <typename T>
__global__ void k_lts_wbar_close(int64_t n, int np6, const uint32_t* mask, const T* zbar, T* wb0, T* wb1, T* wb2,
                                 T* wb3, int nw, double a0, double a1, double a2, double a3) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (lts_row_on(mask, 0, i, np6)) continue;
        const T z = zbar[i];
        if (nw > 0) wb0[i] = (T)a0 * z;
        if (nw > 1) wb1[i] = (T)a1 * z;
        if (nw > 2) wb2[i] = (T)a2 * z;
        if (nw > 3) wb3[i] = (T)a3 * z;
    }
}

__global__ void k_axpby(double a, const double* x, double b, const double* y, double* z, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        z[i] = a * x[i] + b * y[i];
}

template <typename T>
__global__ void k_filter_add(const T* __restrict__ U, double wr, double wi, double* Fre, double* Fim, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double u = (double)U[i];
        Fre[i] += wr * u;
        Fim[i] += wi * u;
    }
}

// F += wa field(U) + wb field(D) (two levels of the filter sum in one pass)
template <typename T>
__global__ void k_filter_add2(const T* __restrict__ U, double ar, double ai, const T* __restrict__ D, double br,
                              double bi, double* Fre, double* Fim, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double u = (double)U[i], d = (double)D[i];
        Fre[i] += ar * u + br * d;
        Fim[i] += ai * u + bi * d;
    }
}

constexpr int kDotBlocks = 1024;
constexpr int kDotThreads = 256;

template <int Q>
__global__ __launch_bounds__(kDotThreads) void k_dot(const double* __restrict__ U, const double* __restrict__ V,
                                                     const double* __restrict__ wE, const double* __restrict__ wH,
                                                     int64_t K, double* __restrict__ partial) {
    constexpr int NP = Dim<Q>::NP;
    constexpr int MMO = mat_off(Q) + 3 * NP * NP + NP * 4 * Dim<Q>::NFP;
    __shared__ double sm[kDotThreads];
    double acc = 0.0;
    const int64_t rows = 6 * K;
    for (int64_t r = blockIdx.x * (int64_t)kDotThreads + threadIdx.x; r < rows; r += (int64_t)gridDim.x * kDotThreads) {
        const double* u = U + r * NP;
        const double* v = V + r * NP;
        double vv[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) vv[j] = v[j];
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            double mvv = 0.0;
#pragma unroll
            for (int j = 0; j < NP; ++j) mvv = fma(cMat64[MMO + i * NP + j], vv[j], mvv);
            s = fma(u[i], mvv, s);
        }
        const int64_t e = r / 6;
        acc = fma(s, (r - 6 * e) < 3 ? wE[e] : wH[e], acc);
    }
    sm[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kDotThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sm[threadIdx.x] += sm[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sm[0];
}

__global__ __launch_bounds__(kDotThreads) void k_dot_final(const double* __restrict__ partial, int n,
                                                           double* __restrict__ out) {
    __shared__ double sm[kDotThreads];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += kDotThreads) acc += partial[i];
    sm[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kDotThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sm[threadIdx.x] += sm[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = sm[0];
}

// Batched dot: member b = blockIdx.y; per member the same block decomposition
// and summation order as k_dot / k_dot_final (results equal the single dots).
template <int Q>
__global__ __launch_bounds__(kDotThreads) void k_dot_batch(const double* __restrict__ U, const double* __restrict__ V,
                                                           const double* __restrict__ wE,
                                                           const double* __restrict__ wH, int64_t wstride,
                                                           int64_t K, double* __restrict__ partial) {
    constexpr int NP = Dim<Q>::NP;
    constexpr int MMO = mat_off(Q) + 3 * NP * NP + NP * 4 * Dim<Q>::NFP;
    __shared__ double sm[kDotThreads];
    const int64_t b = blockIdx.y;
    const int64_t n = 6 * K * NP;
    U += b * n;
    V += b * n;
    wE += b * wstride;
    wH += b * wstride;
    double acc = 0.0;
    const int64_t rows = 6 * K;
    for (int64_t r = blockIdx.x * (int64_t)kDotThreads + threadIdx.x; r < rows; r += (int64_t)gridDim.x * kDotThreads) {
        const double* u = U + r * NP;
        const double* v = V + r * NP;
        double vv[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) vv[j] = v[j];
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            double mvv = 0.0;
#pragma unroll
            for (int j = 0; j < NP; ++j) mvv = fma(cMat64[MMO + i * NP + j], vv[j], mvv);
            s = fma(u[i], mvv, s);
        }
        const int64_t e = r / 6;
        acc = fma(s, (r - 6 * e) < 3 ? wE[e] : wH[e], acc);
    }
    sm[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kDotThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sm[threadIdx.x] += sm[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[b * kDotBlocks + blockIdx.x] = sm[0];
}

__global__ __launch_bounds__(kDotThreads) void k_dot_final_batch(const double* __restrict__ partial, int n,
                                                                 double* __restrict__ out) {
    __shared__ double sm[kDotThreads];
    const int b = blockIdx.x;
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += kDotThreads) acc += partial[(int64_t)b * kDotBlocks + i];
    sm[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kDotThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sm[threadIdx.x] += sm[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[b] = sm[0];
}

__global__ void k_axpby_batch(const double* __restrict__ a, const double* x, const double* __restrict__ c,
                              const double* y, double* z, int64_t n, int B) {
    const int64_t tot = n * B;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < tot; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = i / n;
        z[i] = a[b] * x[i] + c[b] * y[i];
    }
}

template <typename T>
__global__ void k_filter_add_batch(const T* __restrict__ U, const double* __restrict__ wr,
                                   const double* __restrict__ wi, double* Fre, double* Fim, int64_t n, int B) {
    const int64_t tot = n * B;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < tot; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = i / n;
        const double u = (double)U[i];
        Fre[i] += wr[b] * u;
        Fim[i] += wi[b] * u;
    }
}

__global__ void k_nonfinite(const double* X, int64_t n, int* flag) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double x = X[i];
        if (!(x == x) || x - x != 0.0) flag[0] = 1;
    }
}

// Stage-kernel variant per (q, precision): 0 = gather per face, 1 = gathers
// pipelined one face ahead; from 2 on (q >= 2) on the matrix cores, one kernel
// per precision whatever the number: k_stage_col (FP32), k_stage_tile (FP64);
// -1 = chosen per launch from its size.  Overridable through cmcg_tune_stage()
// and the autotuner.  Defaults: per-face gathers for P1, the matrix cores for P2
// and P3, ahead of the VALU form at every size (FP32 P2: 196608 tets 50 / 53 us,
// 64 members of 10368 184 / 200; FP64 P2: 82944 tets 38.5 / 54; P3: 48000 tets
// 50.5 / 116).  The numbers by size are what cmcg_tune_resolve_stage has always
// reported.
int g_variant[kMaxQ + 1][2] = {{0, 0}, {0, 0}, {-1, -1}, {-1, -1}};
inline int variant_by_size(int q, int precision, int64_t blocks) {
    if (precision == CMCG_FP64) {
        if (blocks <= 400) return 9;
        return blocks <= 1100 || (q == 3 && blocks <= 9000) ? 8 : 4;
    }
    if (q == 3) return blocks <= 1100 ? 9 : blocks <= 9000 ? 6 : 4;
    if (q == 2) return blocks <= 1100 ? 9 : blocks <= 3000 ? 5 : blocks <= 12000 ? 4 : 3;
    return 0;
}
inline int stage_variant(int q, int precision, int64_t blocks) {
    const int v = g_variant[q][precision];
    return v >= 0 ? v : variant_by_size(q, precision, blocks);
}

inline int grid_for(int64_t n, int threads = 256) {
    int64_t g = (n + threads - 1) / threads;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    return (int)g;
}

// Grid of k_stage_tile.  P3, single problems: what the device holds at once
// (occ workgroups per compute unit, 32 compute units per XCD), each running
// several blocks where there are more.  Batches: twice as many, dealt out on
// the device to the members that take the step, so that members which have
// converged or have fewer steps leave no part of the device idle; the second
// round evens out what the division leaves over.  A fixed share per member
// against this (ms a solve): 16 members of 10368 tets 366 / 366, one of them with
// six times the steps 1340 / 550; 64 of 3072 397 / 338, 1428 / 404.  Three or four
// rounds cost 1-6 % (the matrix table is read by more workgroups).
template <int Q> inline dim3 tile_grid(int64_t per, unsigned members, int occ) {
    if (!TileDim<Q>::LOOP) return dim3((unsigned)(8 * per), members);
    const int64_t n = per * members, held = 32 * occ;
    const int64_t most = members == 1 ? held : 2 * held > members ? 2 * held : members;
    return dim3((unsigned)(8 * (n < most ? n : most)));
}

// Non-temporal hints for what the update pass reads and writes once per launch,
// where the vectors of a launch exceed the 256 MB Infinity Cache by so much that
// it holds little of them anyway: the stage input's planes, whose face traces
// the neighbouring blocks read, then stay in the caches.  With and without (us
// per launch): FP32 P2 279936 tets (302 MB) 83.4 / 84.5, 384000 (415 MB) 105.9 /
// 111.0, P3 162000 (350 MB) 112.5 / 114.1, 196608 (425 MB) 131.9 / 134.8, FP64 P2
// 196608 (377 MB) 111 / 117, FP64 P3 82944 (319 MB) 94.1 / 95.6; below the line the
// hint sends to memory what the cache would have held: FP32 P2 196608 (212 MB)
// 55.6 / 49.1, P3 48000 (104 MB) 34.3 / 30.6, 131712 (284 MB) 91.6 / 85.5, FP64 P3
// 48000 (184 MB) 55.0 / 50.0.  The filter's
// accumulators (16 B per value, read and written once per step) count as vectors
// of their own; a filtered launch of P2 384000 tets takes 265 us, 142 of them for
// 737 MB of accumulators, a copy's rate (scalar accesses without the hint: 360 us).
template <typename T, int Q> int stream_hints(const StageArgs& a) {  // 2: all, 1: the filter alone
    constexpr double kLine = 300e6;
    // members whose period is over keep their vectors out of it
    const int members = a.nrun > 0 ? a.nrun : a.nmembers > 1 ? a.nmembers : 1;
    const double dofs = (double)a.K * 6 * Dim<Q>::NP * members;
    const double vectors = dofs * (sizeof(T) == 4 ? 18 : 32);  // U, Y, Y', Acc, FP32's low parts
    return vectors > kLine ? 2 : a.filter && vectors + 16 * dofs > kLine ? 1 : 0;
}

template <int Q, bool MH, int STREAM>
void stage_launch_mfma(const StageArgs& a, dim3 grid, int64_t per, int precision, hipStream_t s) {
    if (precision == CMCG_FP32)
        hipLaunchKernelGGL((k_stage_col<Q, MH, false, STREAM>), grid, dim3(ColDim<Q>::NTH), 0, s, a, per);
    else if (TileDim<Q>::LOOP && !MH && a.mtab)  // batches have one frequency
        hipLaunchKernelGGL((k_stage_tile<Q, MH, false, STREAM, TileDim<Q>::LOOP && !MH>),
                           tile_grid<Q>(per, grid.y, TileDim<Q>::occ(false)), dim3(256), 0, s, a, per);
    else
        hipLaunchKernelGGL((k_stage_tile<Q, MH, false, STREAM>), tile_grid<Q>(per, grid.y, TileDim<Q>::occ(false)),
                           dim3(256), 0, s, a, per);
}

template <typename T, int Q, bool MH>
void stage_launch_mh(const StageArgs& a, hipStream_t s) {
    const int64_t blocks = a.blist ? a.nblist : (a.K + EPW - 1) / EPW;
    const int64_t per = (blocks + 7) / 8;
    const int v = stage_variant(Q, sizeof(T) == 8 ? CMCG_FP64 : CMCG_FP32, blocks * (a.nmembers > 1 ? a.nmembers : 1));
    const dim3 grid((unsigned)(8 * per), (unsigned)(a.nmembers > 1 ? a.nmembers : 1));
    if constexpr (Q >= 2) {
        if (v >= 2 && (Q == 3 || (v != 6 && v != 7))) {
            const int prec = sizeof(T) == 8 ? CMCG_FP64 : CMCG_FP32;
            const int hints = MH ? 0 : stream_hints<T, Q>(a);
            if (hints == 0)
                stage_launch_mfma<Q, MH, 0>(a, grid, per, prec, s);
            else if (hints == 1)
                stage_launch_mfma<Q, false, 1>(a, grid, per, prec, s);
            else
                stage_launch_mfma<Q, false, 2>(a, grid, per, prec, s);
            return;
        }
    }
    if (v == 1)
        hipLaunchKernelGGL((k_stage<T, Q, true, MH>), grid, dim3(64), 0, s, a, per);
    else
        hipLaunchKernelGGL((k_stage<T, Q, false, MH>), grid, dim3(64), 0, s, a, per);
}

template <typename T, int Q>
void stage_launch(const StageArgs& a, hipStream_t s) {
    if (a.mode == LTS_FWD || a.mode == LTS_ADJ || a.mode == LTS_CHAIN) {  // one instantiation per order
        const int64_t blocks = a.blist ? a.nblist : (a.K + EPW - 1) / EPW;
        const int64_t per = (blocks + 7) / 8;
        const dim3 grid((unsigned)(8 * per));
        if constexpr (Q >= 2 && std::is_same<T, float>::value)
            hipLaunchKernelGGL((k_stage_col<Q, false, true, 0>), grid, dim3(ColDim<Q>::NTH), 0, s, a, per);
        else if constexpr (Q >= 2)
            hipLaunchKernelGGL((k_stage_tile<Q, false, true, 0>), tile_grid<Q>(per, 1, TileDim<Q>::occ(true)), dim3(256), 0, s, a, per);
        else
            hipLaunchKernelGGL((k_stage<T, Q, false, false, true>), grid, dim3(64), 0, s, a, per);
        return;
    }
    if (a.nharm > 1)
        stage_launch_mh<T, Q, true>(a, s);
    else
        stage_launch_mh<T, Q, false>(a, s);
}

void check_launch() {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) fail(CMCG_ERR_DEVICE, std::string("kernel launch: ") + hipGetErrorString(e));
}

// Fixed device array for the partial sums of the allocation-free inner
// product (one copy per GPU, held until the process ends).  Host code never
// passes its name to a kernel: the name is a host-side stand-in, and the
// device address comes from hipGetSymbolAddress, resolved once per device.
constexpr int kNoallocDoubles = 1024;
static_assert(kNoallocDoubles >= kDotBlocks, "the scratch array must hold every partial of a dot");
__device__ __align__(256) double scratch[kNoallocDoubles];

std::mutex g_scratch_mu;
double* g_scratch_ptr[64] = {};

}  // namespace

size_t noalloc_scratch_doubles() { return kNoallocDoubles; }

double* noalloc_scratch(int device) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (device < 0 || device >= 64) fail(CMCG_ERR_DEVICE, "device index out of range");
    if (!g_scratch_ptr[device]) {
        int cur = -1;
        CMCG_HIP(hipGetDevice(&cur));
        if (cur != device) fail(CMCG_ERR_STATE, "scratch address requested for a device that is not current");
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            (void)hipGetLastError();
            fail(CMCG_ERR_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        }
        g_scratch_ptr[device] = (double*)ptr;
    }
    return g_scratch_ptr[device];
}

int dot_blocks(int64_t K) {
    const int64_t rows = 6 * K;
    int64_t blocks = (rows + kDotThreads - 1) / kDotThreads;
    if (blocks > kDotBlocks) blocks = kDotBlocks;
    return (int)(blocks < 1 ? 1 : blocks);
}

void upload_constants(int q, int precision, const double* D, const double* LIFT, const double* M,
                      const int* fnode, const int* fperm) {
    (void)precision;
    const int NP = np_of(q), NFP = nfp_of(q);
    const int n = mat_size(q);
    std::vector<double> buf(n);
    std::copy(D, D + 3 * NP * NP, buf.begin());
    std::copy(LIFT, LIFT + NP * 4 * NFP, buf.begin() + 3 * NP * NP);
    std::copy(M, M + NP * NP, buf.begin() + 3 * NP * NP + 4 * NP * NFP);
    std::vector<float> bf(buf.begin(), buf.end());
    const size_t off = mat_off(q);
    CMCG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(cMat64), buf.data(), n * sizeof(double), off * sizeof(double),
                               hipMemcpyHostToDevice));
    CMCG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(cMat32), bf.data(), n * sizeof(float), off * sizeof(float),
                               hipMemcpyHostToDevice));
    {
        std::vector<int> nn(24 * NFP);
        for (int nf = 0; nf < 4; ++nf)
            for (int pm = 0; pm < 6; ++pm)
                for (int k = 0; k < NFP; ++k) nn[(nf * 6 + pm) * NFP + k] = fnode[nf * NFP + fperm[pm * NFP + k]];
        std::vector<uint32_t> words(ft_words(q), 0u);
        for (int i = 0; i < 28 * NFP; ++i) {
            const int v = i < 4 * NFP ? fnode[i] : nn[i - 4 * NFP];
            if (v < 0 || v > 255) fail(CMCG_ERR_ARG, "face-node table entry out of byte range");
            words[i / 4] |= (uint32_t)v << (8 * (i % 4));
        }
        CMCG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(cFaceTab), words.data(), words.size() * sizeof(uint32_t),
                                   ft_off(q) * sizeof(uint32_t), hipMemcpyHostToDevice));
    }
    if (q >= 2) {
        // broadcast operands of the FP32 kernels with one column per lane (gCol)
        const int W = (NP + 3) / 4, NV = (3 * NP + 15) / 16, NL = (4 * NFP + 15) / 16;
        std::vector<float> t((size_t)W * (NV + NL) * 64, 0.f);
        for (int w = 0; w < W; ++w)
            for (int l = 0; l < 64; ++l) {
                const int i = 4 * w + l % 4;
                if (i >= NP) continue;
                float* o = &t[(size_t)w * (NV + NL) * 64 + l];
                for (int v = 0; v < NV; ++v) {
                    const int st = 16 * v + l / 4;
                    if (st < 3 * NP) o[64 * v] = (float)D[(st % 3 * NP + i) * NP + st / 3];
                }
                for (int v = 0; v < NL; ++v) {
                    const int st = 16 * v + l / 4;
                    if (st < 4 * NFP) o[64 * (NV + v)] = (float)LIFT[i * 4 * NFP + st];
                }
            }
        CMCG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(gCol), t.data(), t.size() * sizeof(float), col_off(q) * sizeof(float),
                                   hipMemcpyHostToDevice));
    }
    if (q >= 2) {
        // A operands of the FP64 kernels' K steps (gTile)
        const int NJ = (NP + 3) / 4, KSV = 3 * NJ, NST = KSV + NFP, tail = NP > 16;
        std::vector<double> t((size_t)NST * (tail ? 80 : 64), 0.0);
        const auto at = [&](int i, int st, int k) {  // row i, K row k of step st
            if (i >= NP) return 0.0;
            if (st >= KSV) return LIFT[i * 4 * NFP + 4 * (st - KSV) + k];
            const int j = 4 * (st % NJ) + k;
            return j < NP ? D[(st / NJ * NP + i) * NP + j] : 0.0;
        };
        for (int st = 0; st < NST; ++st) {
            for (int l = 0; l < 64; ++l) t[st * 64 + l] = at(l % 16, st, l / 16);
            for (int l = 0; tail && l < 16; ++l) t[NST * 64 + st * 16 + l] = at(16 + l % 4, st, l / 4);
        }
        CMCG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(gTile), t.data(), t.size() * sizeof(double),
                                   (q == 2 ? 0 : TileDim<2>::NTAB) * sizeof(double), hipMemcpyHostToDevice));
    }
}

void launch_stage(int q, int precision, const StageArgs& a, hipStream_t s) {
    if (precision == CMCG_FP64) {
        if (q == 1) stage_launch<double, 1>(a, s);
        else if (q == 2) stage_launch<double, 2>(a, s);
        else stage_launch<double, 3>(a, s);
    } else {
        if (q == 1) stage_launch<float, 1>(a, s);
        else if (q == 2) stage_launch<float, 2>(a, s);
        else stage_launch<float, 3>(a, s);
    }
    check_launch();
}

namespace {
template <typename F> auto period_kernel(int q, int precision, F f) {
    if (precision == CMCG_FP64) {
        if (q == 1) return f(k_period_p1<double>, 256);
        return q == 2 ? f(k_period_tile<2, 3>, 256) : f(k_period_tile<3, 2>, 256);
    }
    if (q == 1) return f(k_period_p1<float>, 256);
    return q == 2 ? f(k_period_col<2, 4>, ColDim<2>::NTH) : f(k_period_col<3, 5>, ColDim<3>::NTH);
}
}  // namespace

int64_t period_room(int q, int precision) {
    return period_kernel(q, precision, [](auto kernel, int threads) { return resident_room(kernel, threads); });
}

void launch_period(int q, int precision, const PeriodArgs& a, int n, int left_out, hipStream_t s) {
    period_kernel(q, precision, [&](auto kernel, int threads) {
        launch_resident(kernel, (a.K + EPW - 1) / EPW, n, left_out, threads, a, s);
    });
}

void launch_to_field(int precision, int Np, const double* X, void* U, void* Ulo, int64_t n, int flipH,
                     hipStream_t s) {
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_to_field<double>, dim3(grid_for(n)), dim3(256), 0, s, X, (double*)U, nullptr, n, Np,
                           flipH);
    else
        hipLaunchKernelGGL(k_to_field<float>, dim3(grid_for(n)), dim3(256), 0, s, X, (float*)U, (uint16_t*)Ulo, n,
                           Np, flipH);
    check_launch();
}

void launch_from_field(int precision, int Np, const void* U, const void* Ulo, double* Y, const double* sub,
                       int64_t n, int flipH, hipStream_t s) {
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_from_field<double>, dim3(grid_for(n)), dim3(256), 0, s, (const double*)U, nullptr, Y,
                           sub, n, Np, flipH);
    else
        hipLaunchKernelGGL(k_from_field<float>, dim3(grid_for(n)), dim3(256), 0, s, (const float*)U,
                           (const uint16_t*)Ulo, Y, sub, n, Np, flipH);
    check_launch();
}

void launch_copy_field(int precision, const void* src, void* dst, int64_t n, hipStream_t s) {
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_copy<double>, dim3(grid_for(n)), dim3(256), 0, s, (const double*)src, (double*)dst, n);
    else
        hipLaunchKernelGGL(k_copy<float>, dim3(grid_for(n)), dim3(256), 0, s, (const float*)src, (float*)dst, n);
    check_launch();
}

void launch_zero(void* p, size_t bytes, hipStream_t s) {
    const int64_t n = (int64_t)(bytes / 4);
    hipLaunchKernelGGL(k_zero, dim3(grid_for(n)), dim3(256), 0, s, (uint32_t*)p, n);
    check_launch();
}

int64_t source_mask_words(int64_t K) { return (K + EPW - 1) / EPW; }

void launch_source_mask(int precision, int Np, const void* Sre, const void* Sim, int nharm, int64_t hstride,
                        int64_t K, uint32_t* mask, hipStream_t s) {
    const int64_t nb = source_mask_words(K);
    if (nb == 0) return;
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_source_mask<double>, dim3((unsigned)nb), dim3(64), 0, s, (const double*)Sre,
                           (const double*)Sim, nharm, hstride, K, 6 * Np, mask);
    else
        hipLaunchKernelGGL(k_source_mask<float>, dim3((unsigned)nb), dim3(64), 0, s, (const float*)Sre,
                           (const float*)Sim, nharm, hstride, K, 6 * Np, mask);
    check_launch();
}

void launch_axpby(double a, const double* x, double b, const double* y, double* z, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_axpby, dim3(grid_for(n)), dim3(256), 0, s, a, x, b, y, z, n);
    check_launch();
}

void launch_filter_add(int precision, const void* U, double wr, double wi, double* Fre, double* Fim, int64_t n,
                       hipStream_t s) {
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_filter_add<double>, dim3(grid_for(n)), dim3(256), 0, s, (const double*)U, wr, wi, Fre,
                           Fim, n);
    else
        hipLaunchKernelGGL(k_filter_add<float>, dim3(grid_for(n)), dim3(256), 0, s, (const float*)U, wr, wi, Fre,
                           Fim, n);
    check_launch();
}

void launch_filter_add2(int precision, const void* U, double ar, double ai, const void* D, double br, double bi,
                        double* Fre, double* Fim, int64_t n, hipStream_t s) {
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_filter_add2<double>, dim3(grid_for(n)), dim3(256), 0, s, (const double*)U, ar, ai,
                           (const double*)D, br, bi, Fre, Fim, n);
    else
        hipLaunchKernelGGL(k_filter_add2<float>, dim3(grid_for(n)), dim3(256), 0, s, (const float*)U, ar, ai,
                           (const float*)D, br, bi, Fre, Fim, n);
    check_launch();
}

int dot_partials() { return kDotBlocks; }

namespace {
LtsRange lts_range(int64_t n, int np6, const int* blist, int64_t nb) {
    LtsRange r;
    r.blist = blist;
    r.nb = nb;
    r.n = n;
    r.per = (int64_t)EPW * np6;
    return r;
}
int64_t lts_count(const LtsRange& r) { return r.blist ? r.nb * r.per : r.n; }
}  // namespace

void launch_lts_axpy(int precision, int64_t n, int np6, const int* blist, int64_t nb, const uint32_t* mask, int inv,
                     double a, const void* y, double b, const void* x, void* z, hipStream_t s) {
    const LtsRange rg = lts_range(n, np6, blist, nb);
    const int g = grid_for(lts_count(rg));
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_lts_axpy<double>, dim3(g), dim3(256), 0, s, rg, np6, mask, inv, a, (const double*)y,
                           b, (const double*)x, (double*)z);
    else
        hipLaunchKernelGGL(k_lts_axpy<float>, dim3(g), dim3(256), 0, s, rg, np6, mask, inv, a, (const float*)y, b,
                           (const float*)x, (float*)z);
    check_launch();
}

void launch_lts_closed(int precision, int64_t n, int np6, int Np, const uint32_t* mask, const void* const* W,
                       const double* al, int nw, const void* Sre, const void* Sim, int src_rows, double sc, double ss,
                       void* z, hipStream_t s) {
    const void* Wp[4] = {nullptr, nullptr, nullptr, nullptr};
    double c[4] = {0, 0, 0, 0};
    for (int j = 0; j < nw && j < 4; ++j) {
        Wp[j] = W[j];
        c[j] = al[j];
    }
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_lts_closed<double>, dim3(grid_for(n)), dim3(256), 0, s, n, np6, Np, mask,
                           (const double*)Wp[0], (const double*)Wp[1], (const double*)Wp[2], (const double*)Wp[3], nw,
                           c[0], c[1], c[2], c[3], (const double*)Sre, (const double*)Sim, src_rows, sc, ss,
                           (double*)z);
    else
        hipLaunchKernelGGL(k_lts_closed<float>, dim3(grid_for(n)), dim3(256), 0, s, n, np6, Np, mask,
                           (const float*)Wp[0], (const float*)Wp[1], (const float*)Wp[2], (const float*)Wp[3], nw,
                           c[0], c[1], c[2], c[3], (const float*)Sre, (const float*)Sim, src_rows, sc, ss,
                           (float*)z);
    check_launch();
}

void launch_lts_wbar_close(int precision, int64_t n, int np6, const uint32_t* mask, const void* zbar,
                           void* const* wb, const double* al, int nw, hipStream_t s) {
    void* W[4] = {nullptr, nullptr, nullptr, nullptr};
    double c[4] = {0, 0, 0, 0};
    for (int j = 0; j < nw && j < 4; ++j) {
        W[j] = wb[j];
        c[j] = al[j];
    }
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_lts_wbar_close<double>, dim3(grid_for(n)), dim3(256), 0, s, n, np6, mask,
                           (const double*)zbar, (double*)W[0], (double*)W[1], (double*)W[2], (double*)W[3], nw, c[0],
                           c[1], c[2], c[3]);
    else
        hipLaunchKernelGGL(k_lts_wbar_close<float>, dim3(grid_for(n)), dim3(256), 0, s, n, np6, mask,
                           (const float*)zbar, (float*)W[0], (float*)W[1], (float*)W[2], (float*)W[3], nw, c[0], c[1],
                           c[2], c[3]);
    check_launch();
}

void launch_mfma_probe(int precision, const double* A, const double* B, double* D, hipStream_t s) {
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_mfma_probe<double>, dim3(1), dim3(64), 0, s, A, B, D);
    else
        hipLaunchKernelGGL(k_mfma_probe<float>, dim3(1), dim3(64), 0, s, A, B, D);
    check_launch();
}

void set_stage_variant(int q, int precision, int variant) { g_variant[q][precision] = variant; }
int get_stage_variant(int q, int precision) { return g_variant[q][precision]; }
int resolve_stage_variant(int q, int precision, int64_t K, int members) {
    if (q < 1 || q > kMaxQ) return 0;
    return stage_variant(q, precision, (K + EPW - 1) / EPW * (members > 1 ? members : 1));
}

void launch_dot(int q, const double* U, const double* V, const double* wE, const double* wH, int64_t K,
                double* partial, double* out_dev, hipStream_t s) {
    const int blocks = dot_blocks(K);
    if (q == 1)
        hipLaunchKernelGGL(k_dot<1>, dim3(blocks), dim3(kDotThreads), 0, s, U, V, wE, wH, K, partial);
    else if (q == 2)
        hipLaunchKernelGGL(k_dot<2>, dim3(blocks), dim3(kDotThreads), 0, s, U, V, wE, wH, K, partial);
    else
        hipLaunchKernelGGL(k_dot<3>, dim3(blocks), dim3(kDotThreads), 0, s, U, V, wE, wH, K, partial);
    check_launch();
    hipLaunchKernelGGL(k_dot_final, dim3(1), dim3(kDotThreads), 0, s, partial, blocks, out_dev);
    check_launch();
}

void launch_dot_batch(int q, const double* U, const double* V, const double* wE, const double* wH, int64_t wstride,
                      int64_t K, int B, double* partial, double* out_dev, hipStream_t s) {
    int64_t rows = 6 * K;
    int blocks = (int)((rows + kDotThreads - 1) / kDotThreads);
    if (blocks > kDotBlocks) blocks = kDotBlocks;
    const dim3 grid(blocks, B);
    if (q == 1)
        hipLaunchKernelGGL(k_dot_batch<1>, grid, dim3(kDotThreads), 0, s, U, V, wE, wH, wstride, K, partial);
    else if (q == 2)
        hipLaunchKernelGGL(k_dot_batch<2>, grid, dim3(kDotThreads), 0, s, U, V, wE, wH, wstride, K, partial);
    else
        hipLaunchKernelGGL(k_dot_batch<3>, grid, dim3(kDotThreads), 0, s, U, V, wE, wH, wstride, K, partial);
    check_launch();
    hipLaunchKernelGGL(k_dot_final_batch, dim3(B), dim3(kDotThreads), 0, s, partial, blocks, out_dev);
    check_launch();
}

void launch_axpby_batch(const double* a, const double* x, const double* c, const double* y, double* z, int64_t n,
                        int B, hipStream_t s) {
    hipLaunchKernelGGL(k_axpby_batch, dim3(grid_for(n * B)), dim3(256), 0, s, a, x, c, y, z, n, B);
    check_launch();
}

void launch_filter_add_batch(int precision, const void* U, const double* w_re, const double* w_im, double* Fre,
                             double* Fim, int64_t n, int B, hipStream_t s) {
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_filter_add_batch<double>, dim3(grid_for(n * B)), dim3(256), 0, s, (const double*)U,
                           w_re, w_im, Fre, Fim, n, B);
    else
        hipLaunchKernelGGL(k_filter_add_batch<float>, dim3(grid_for(n * B)), dim3(256), 0, s, (const float*)U,
                           w_re, w_im, Fre, Fim, n, B);
    check_launch();
}

void launch_nonfinite(const double* X, int64_t n, int* out_dev, hipStream_t s) {
    hipLaunchKernelGGL(k_nonfinite, dim3(grid_for(n)), dim3(256), 0, s, X, n, out_dev);
    check_launch();
}

}  // namespace cmcg
