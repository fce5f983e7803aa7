// Kernels of the 2-D transverse-magnetic path (Section 5.2.1, two-dimensional
// setting; Section 5.2.2 DG scheme on triangles; Section 5.3 Runge-Kutta
// stages): fields (e, h1, h2), dof layout [K][3][Np].
//
// Stage kernel: one 64-lane workgroup per block of 21 triangles, lane =
// (triangle, component).  The block's stage input is staged in LDS with one
// coalesced load, together with the order's D and LIFT (read afterwards as
// LDS broadcasts, which shortens the chain of scalar-cache loads a lone wave
// otherwise waits on); each lane differentiates its own component, and the
// curl terms are exchanged between the three lanes of a triangle:
//   e row:  -scurl h = -(d1 h2 - d2 h1),   h1 row: d2 e,   h2 row: -d1 e.
// The upwind flux of the lane's component is formed at the Nfp nodes of each
// edge (own traces from LDS, neighbour traces from the field) and lifted with
// LIFT.  The Runge-Kutta update, the compensated FP32 state and the filter
// accumulation follow the stage modes of launch.h, as in the 3-D kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>
#include <type_traits>
#include <vector>

#include "internal.h"
#include "launch.h"
#include "mfma_cols.h"
#include "tagged.h"

namespace cmcg {

namespace {

template <int Q> struct Dim2 {
    static constexpr int NP = (Q + 1) * (Q + 2) / 2;
    static constexpr int NFP = Q + 1;
    static constexpr int MAT = 2 * NP * NP + NP * 3 * NFP + NP * NP;  // D | LIFT | M
};
constexpr int mat2_off(int q) { return q <= 1 ? 0 : q == 2 ? Dim2<1>::MAT : Dim2<1>::MAT + Dim2<2>::MAT; }
constexpr int kMat2Total = Dim2<1>::MAT + Dim2<2>::MAT + Dim2<3>::MAT;

__constant__ double c2Mat64[kMat2Total];
__constant__ float c2Mat32[kMat2Total];

template <typename T> __device__ __forceinline__ const T* mats2();
template <> __device__ __forceinline__ const double* mats2<double>() { return c2Mat64; }
template <> __device__ __forceinline__ const float* mats2<float>() { return c2Mat32; }

constexpr int EPB = 21;  // triangles per 64-lane workgroup (63 active lanes)
constexpr int64_t kEarlyBlocks = 2048;

// Element node of edge node k of edge f (nodes (i, j)/q, j slowest; edge 0 runs
// from vertex 1 to vertex 2, edge 1 from 0 to 2, edge 2 from 0 to 1).
template <int Q> __device__ __host__ constexpr int edge_node(int f, int k) {
    // node (i, j) has index j (Q + 1) - j (j - 1) / 2 + i
    return f == 0 ? k * (Q + 1) - k * (k - 1) / 2 + (Q - k) : f == 1 ? k * (Q + 1) - k * (k - 1) / 2 : k;
}

__device__ __forceinline__ uint16_t to_bf16(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint32_t h) { return __uint_as_float(h << 16); }

// NP contiguous values of one row in pairs: 8-byte accesses for FP32 rows,
// 16-byte for FP64 rows, when rows start on such boundaries (they start at
// multiples of NP sizeof(T) bytes: P2 and P3), single accesses otherwise;
// bfloat16 rows likewise in 4-byte pairs.
template <typename T, int NP> struct Row2 {
    static constexpr bool V2 = NP % 2 == 0;
    using P2 = typename std::conditional<sizeof(T) == 4, float2, double2>::type;
    __device__ __forceinline__ static void load(const T* __restrict__ p, T (&r)[NP]) {
        if constexpr (V2) {
            const P2* q = reinterpret_cast<const P2*>(p);
#pragma unroll
            for (int c = 0; c < NP / 2; ++c) {
                const P2 v = q[c];
                r[2 * c] = v.x;
                r[2 * c + 1] = v.y;
            }
        } else {
#pragma unroll
            for (int i = 0; i < NP; ++i) r[i] = p[i];
        }
    }
    __device__ __forceinline__ static void store(T* __restrict__ p, const T (&r)[NP]) {
        if constexpr (V2) {
            P2* q = reinterpret_cast<P2*>(p);
#pragma unroll
            for (int c = 0; c < NP / 2; ++c) {
                P2 v;
                v.x = r[2 * c];
                v.y = r[2 * c + 1];
                q[c] = v;
            }
        } else {
#pragma unroll
            for (int i = 0; i < NP; ++i) p[i] = r[i];
        }
    }
};
template <int NP> struct RowLo2 {
    static constexpr bool V2 = (NP * 2) % 4 == 0;
    __device__ __forceinline__ static void load(const uint16_t* __restrict__ p, float (&r)[NP]);
    __device__ __forceinline__ static void store(uint16_t* __restrict__ p, const float (&r)[NP]);
};
template <int NP>
__device__ __forceinline__ void RowLo2<NP>::load(const uint16_t* __restrict__ p, float (&r)[NP]) {
    if constexpr (V2) {
        const uint32_t* q = reinterpret_cast<const uint32_t*>(p);
#pragma unroll
        for (int c = 0; c < NP / 2; ++c) {
            const uint32_t w = q[c];
            r[2 * c] = __uint_as_float(w << 16);
            r[2 * c + 1] = __uint_as_float(w & 0xffff0000u);
        }
    } else {
#pragma unroll
        for (int i = 0; i < NP; ++i) r[i] = __uint_as_float((uint32_t)p[i] << 16);
    }
}

template <int NP>
__device__ __forceinline__ void RowLo2<NP>::store(uint16_t* __restrict__ p, const float (&r)[NP]) {
    if constexpr (V2) {
        uint32_t* q = reinterpret_cast<uint32_t*>(p);
#pragma unroll
        for (int c = 0; c < NP / 2; ++c) q[c] = (uint32_t)to_bf16(r[2 * c]) | ((uint32_t)to_bf16(r[2 * c + 1]) << 16);
    } else {
#pragma unroll
        for (int i = 0; i < NP; ++i) p[i] = to_bf16(r[i]);
    }
}

__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e) {
    s = a + b;
    const float bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// Arguments of this workgroup's member in a batched launch (grid.y = member):
// field, geometry and source pointers move by whole members, the stage
// scalars come from the member table; false when the member is idle (its CG
// has converged, or its period has fewer steps than this launch's).
template <typename T>
__device__ __forceinline__ bool member_args2d(const StageArgs& in, StageArgs& a) {
    a = in;
    a.smask = nullptr;
    if (!in.mtab) return true;
    const int b = blockIdx.y;
    if (!in.active[b]) return false;
    if (in.step >= 0 && in.step >= in.msteps[b]) return false;
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
    return true;
}

// The arithmetic shared by the stage and the period kernel is written with
// explicit fma(): left to the compiler, the two contracted the same
// expressions differently and their results parted in the last bit.
//
// Upwind flux (e, h1, h2) at one edge node, g = the edge's normal and flux
// coefficients.
template <typename T>
__device__ __forceinline__ void upwind2d(const T* g, T em, T h1m, T h2m, T ep, T h1p, T h2p, T (&fl)[3]) {
    const T n0 = g[0], n1 = g[1];
    const T cE1 = g[2], cE2 = g[3], cH1 = g[4], cH2 = g[5];
    const T de = ep - em, dh1 = h1p - h1m, dh2 = h2p - h2m;
    const T ndh = fma(n0, dh1, n1 * dh2);
    fl[0] = fma(cE1, de, -cE2 * fma(n0, dh2, -n1 * dh1));
    fl[1] = fma(cH1, fma(-ndh, n0, dh1), cH2 * (n1 * de));
    fl[2] = fma(cH1, fma(-ndh, n1, dh2), -cH2 * (n0 * de));
}

template <typename T, int Q, bool EARLY>
__global__ __launch_bounds__(64) void k_stage2d(StageArgs args, int64_t per) {
    constexpr int NP = Dim2<Q>::NP, NFP = Dim2<Q>::NFP, NF3 = 3 * NFP;
    constexpr int MO = 0;                 // D [2][NP][NP] in sM
    constexpr int LO = 2 * NP * NP;       // LIFT [NP][3 NFP] in sM
    constexpr int NM = 2 * NP * NP + NP * NF3;
    constexpr int ROWS = EPB * 3;
    __shared__ __align__(16) T sY[ROWS * NP];
    __shared__ __align__(16) T sG[EPB * kGeo2];
    __shared__ int sC[EPB * 3];
    __shared__ T sM[NM];  // the order's D and LIFT, read as LDS broadcasts

    StageArgs a;
    if (!member_args2d<T>(args, a)) return;  // uniform per workgroup
    const int64_t b = blockIdx.x;
    const int64_t blk = (b & 7) * per + (b >> 3);  // consecutive blocks on one XCD
    const int64_t e0 = blk * EPB;
    if (e0 >= a.K) return;
    const int lane = threadIdx.x;
    const int ne = (int)((a.K - e0) < EPB ? (a.K - e0) : EPB);
    const T* __restrict__ Y = (const T*)a.Y;
    const T* __restrict__ geo = (const T*)a.geo;
    {
        // every staging load is issued before the first is consumed (loops of
        // a compile-time trip count; a loop that stored each value as it
        // arrived waited for one load at a time), then written to LDS.  The
        // stage input goes in pairs when the chunk starts on a pair boundary
        // and holds whole pairs, the geometry records (28 values) in 16-byte
        // groups.
        constexpr int PV = Row2<T, NP>::V2 ? 2 : 1;
        constexpr int GV = 16 / (int)sizeof(T);
        // native vectors: arrays of them stay in registers
        typedef T VY __attribute__((ext_vector_type(PV)));
        typedef T VG __attribute__((ext_vector_type(GV)));
        static_assert(kGeo2 % GV == 0, "geometry records split into 16-byte groups");
        constexpr int NYL = (EPB * 3 * NP / PV + 63) / 64, NGL = (EPB * kGeo2 / GV + 63) / 64;
        constexpr int NML = (NM + 63) / 64, NCL = (EPB * 3 + 63) / 64;
        const int nyl = ne * 3 * NP / PV, ngl = ne * kGeo2 / GV;
        const VY* ys = reinterpret_cast<const VY*>(Y + e0 * 3 * NP);
        const VG* gs = reinterpret_cast<const VG*>(geo + e0 * kGeo2);
        const T* gm = mats2<T>() + mat2_off(Q);
        VY ry[NYL];
        VG rg[NGL];
        T rm[NML];
        int rc[NCL];
#pragma unroll
        for (int i = 0; i < NYL; ++i)
            if (lane + 64 * i < nyl) ry[i] = ys[lane + 64 * i];
#pragma unroll
        for (int i = 0; i < NGL; ++i)
            if (lane + 64 * i < ngl) rg[i] = gs[lane + 64 * i];
#pragma unroll
        for (int i = 0; i < NCL; ++i)
            if (lane + 64 * i < ne * 3) rc[i] = a.conn[e0 * 3 + lane + 64 * i];
#pragma unroll
        for (int i = 0; i < NML; ++i)
            if (lane + 64 * i < NM) rm[i] = gm[lane + 64 * i];
        VY* yd = reinterpret_cast<VY*>(sY);
        VG* gd = reinterpret_cast<VG*>(sG);
#pragma unroll
        for (int i = 0; i < NYL; ++i)
            if (lane + 64 * i < nyl) yd[lane + 64 * i] = ry[i];
#pragma unroll
        for (int i = 0; i < NGL; ++i)
            if (lane + 64 * i < ngl) gd[lane + 64 * i] = rg[i];
#pragma unroll
        for (int i = 0; i < NCL; ++i)
            if (lane + 64 * i < ne * 3) sC[lane + 64 * i] = rc[i];
#pragma unroll
        for (int i = 0; i < NML; ++i)
            if (lane + 64 * i < NM) sM[lane + 64 * i] = rm[i];
    }
    __syncthreads();

    const int el = lane / 3;
    const int c = lane - 3 * el;
    const bool act = el < ne;
    const int elc = act ? el : 0;
    const int row = elc * 3 + c;
    const int64_t grow = (e0 * 3 + row) * NP;
    const int mode = a.mode;
    constexpr bool COMP = std::is_same<T, float>::value;
    const bool needL = COMP && (mode == RK2_S2 || mode == RK4_S4);
    const bool needU = mode == RK2_S2 || mode == RK4_S2 || mode == RK4_S3 || needL;
    const bool needA = mode == RK4_S2 || mode == RK4_S3 || mode == RK4_S4;
    const T* Mt = sM;
    const T* gg = &sG[elc * kGeo2];

    // ---- EARLY: every global load of the stage is requested here, before the
    // volume work (neighbour traces of the three edges, update operands,
    // source rows): for launches of about one wave per SIMD, where each wave's
    // chain of dependent loads sets the time.  Otherwise the traces are
    // gathered per edge and the update operands loaded after the lift, which
    // keeps the registers (and so the occupancy) of large launches in check.
    // Each lane gathers its own component of the neighbour's edge trace; the
    // triangle's three lanes then exchange them (lanes 3 el + c), so every
    // trace value is loaded once.
    const int base = 3 * elc;
    T nv[3][NFP];
    auto gather = [&](int f, T (&own)[NFP]) {
        const int code = sC[elc * 3 + f];
#pragma unroll
        for (int k = 0; k < NFP; ++k) {
            if (code >= 0) {
                const int64_t nb = code >> 5;
                const int nf = (code >> 3) & 3;
                const int kk = (code & 7) ? NFP - 1 - k : k;
                own[k] = Y[nb * 3 * NP + c * NP + edge_node<Q>(nf, kk)];
            } else {
                own[k] = T(0);
            }
        }
    };
    auto expand = [&](const T (&own)[NFP], T (&tr)[NFP][3]) {
#pragma unroll
        for (int k = 0; k < NFP; ++k) {
            tr[k][0] = __shfl(own[k], base);
            tr[k][1] = __shfl(own[k], base + 1);
            tr[k][2] = __shfl(own[k], base + 2);
        }
    };
    T up[NP], ap[NP], sr[NP], si[NP];
    float lo[NP];
    const bool src = act && c < a.src_rows;
    auto operands = [&]() {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            up[i] = ap[i] = sr[i] = si[i] = T(0);
            lo[i] = 0.f;
        }
        if (act && needU) Row2<T, NP>::load((const T*)a.U + grow, up);
        if (act && needA) Row2<T, NP>::load((const T*)a.Acc + grow, ap);
        if (act && needL) RowLo2<NP>::load((const uint16_t*)a.Ulo + grow, lo);
        if (src) {
            Row2<T, NP>::load((const T*)a.Sre + grow, sr);
            Row2<T, NP>::load((const T*)a.Sim + grow, si);
        }
    };
    if constexpr (EARLY) {
#pragma unroll
        for (int f = 0; f < 3; ++f) gather(f, nv[f]);
        operands();
    }

    // ---- volume: physical derivatives of the lane's component
    T y[NP], d1[NP], d2[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) y[j] = sY[row * NP + j];
    const T g00 = gg[0], g01 = gg[1], g10 = gg[2], g11 = gg[3];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        T r0 = T(0), r1 = T(0);
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            r0 = fma(Mt[MO + i * NP + j], y[j], r0);
            r1 = fma(Mt[MO + NP * NP + i * NP + j], y[j], r1);
        }
        d1[i] = fma(g00, r0, g10 * r1);
        d2[i] = fma(g01, r0, g11 * r1);
    }
    // curl exchange between the triangle's lanes (3 el: e, 3 el + 1: h1, 3 el + 2: h2)
    const int srcA = c == 0 ? base + 2 : base;  // lane whose d1 is taken
    const int srcB = c == 0 ? base + 1 : base;  // lane whose d2 is taken
    const T sa = c == 1 ? T(0) : T(-1);
    const T sb = c == 2 ? T(0) : T(1);
    T acc[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        const T A = __shfl(d1[i], srcA);
        const T B = __shfl(d2[i], srcB);
        acc[i] = fma(sa, A, sb * B);
    }

    // ---- upwind flux of the lane's component on each edge, lifted
    auto face = [&](int f, const T (&tr)[NFP][3]) {
        const int code = sC[elc * 3 + f];
        // read once per edge, ahead of the branches below (P3 FP32, 30276 triangles:
        // 9.2 us a launch; read in each branch 9.6)
        T g[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) g[i] = gg[4 + 6 * f + i];
        T fl[NFP];
#pragma unroll
        for (int k = 0; k < NFP; ++k) {
            const int own = edge_node<Q>(f, k);
            const T em = sY[(elc * 3) * NP + own];
            const T h1m = sY[(elc * 3 + 1) * NP + own];
            const T h2m = sY[(elc * 3 + 2) * NP + own];
            T ep = tr[k][0], h1p = tr[k][1], h2p = tr[k][2];
            if (code == -1) {  // PEC ghost: e+ = -e-, h+ = h-
                ep = -em;
                h1p = h1m;
                h2p = h2m;
            }  // impedance ghost (homogeneous part): zero exterior state, as gathered
            T v[3];
            if (c == 0) {  // branches: one component is needed, and selects cost registers
                upwind2d(g, em, h1m, h2m, ep, h1p, h2p, v);
                fl[k] = v[0];
            } else {
                upwind2d(g, em, h1m, h2m, ep, h1p, h2p, v);
                fl[k] = c == 1 ? v[1] : v[2];
            }
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            T t = acc[i];
#pragma unroll
            for (int k = 0; k < NFP; ++k) t = fma(Mt[LO + i * NF3 + f * NFP + k], fl[k], t);
            acc[i] = t;
        }
    };
    if constexpr (EARLY) {
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            T tr[NFP][3];
            expand(nv[f], tr);
            face(f, tr);
        }
    } else {
#pragma unroll 1
        for (int f = 0; f < 3; ++f) {
            T own[NFP], tr[NFP][3];
            gather(f, own);
            expand(own, tr);
            face(f, tr);
        }
    }
    if (!act) return;
    if constexpr (!EARLY) operands();

    // ---- stage update of the lane's row
    const T inv = c == 0 ? gg[22] : gg[23];
    const T sig = c == 0 ? gg[24] : T(0);
    T kv[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) kv[i] = fma(inv, acc[i], -sig * y[i]);
    if (src) {
        const T scos = (T)a.scos, ssin = (T)a.ssin;
#pragma unroll
        for (int i = 0; i < NP; ++i) kv[i] = fma(scos, sr[i], fma(-ssin, si[i], kv[i]));
        // further harmonics of a several-frequency source (single launches only,
        // so the kernel arguments hold this problem's tables; they are indexed
        // there, not in the local copy, which would go to scratch)
#pragma unroll 1
        for (int h = 1; h < args.nharm; ++h) {
            Row2<T, NP>::load((const T*)args.Sre + h * args.hstride + grow, sr);
            Row2<T, NP>::load((const T*)args.Sim + h * args.hstride + grow, si);
            const T hc = (T)args.hcos[h], hs = (T)args.hsin[h];
#pragma unroll
            for (int i = 0; i < NP; ++i) kv[i] += hc * sr[i] - hs * si[i];
        }
    }
    const T cy = (T)a.cy, ca = (T)a.ca, cu = (T)a.cu;
    T o1[NP], o2[NP];
    float lo2[NP];
    switch (mode) {
        case RK2_S1:
#pragma unroll
            for (int i = 0; i < NP; ++i) o1[i] = fma(cy, kv[i], y[i]);
            Row2<T, NP>::store((T*)a.Ynext + grow, o1);
            break;
        case RK2_S2:
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                if constexpr (COMP)
                    two_sum(up[i], fma(cu, kv[i], lo[i]), o1[i], lo2[i]);
                else
                    o1[i] = fma(cu, kv[i], up[i]);
            }
            Row2<T, NP>::store((T*)a.Uout + grow, o1);
            if constexpr (COMP) RowLo2<NP>::store((uint16_t*)a.Ulo + grow, lo2);
            break;
        case RK4_S1:
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                o1[i] = fma(cy, kv[i], y[i]);
                o2[i] = COMP ? ca * kv[i] : fma(ca, kv[i], y[i]);
            }
            Row2<T, NP>::store((T*)a.Ynext + grow, o1);
            Row2<T, NP>::store((T*)a.Acc + grow, o2);
            break;
        case RK4_S2:
        case RK4_S3:
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                o1[i] = fma(cy, kv[i], up[i]);
                o2[i] = fma(ca, kv[i], ap[i]);
            }
            Row2<T, NP>::store((T*)a.Ynext + grow, o1);
            Row2<T, NP>::store((T*)a.Acc + grow, o2);
            break;
        case RK4_S4:
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                if constexpr (COMP)
                    two_sum(up[i], fma(cu, kv[i], ap[i]) + lo[i], o1[i], lo2[i]);
                else
                    o1[i] = fma(cu, kv[i], ap[i]);
            }
            Row2<T, NP>::store((T*)a.Uout + grow, o1);
            if constexpr (COMP) RowLo2<NP>::store((uint16_t*)a.Ulo + grow, lo2);
            break;
        default:
            Row2<T, NP>::store((T*)a.Kout + grow, kv);
            break;
    }
    if (a.filter) {
        double* fr = a.Fre + grow;
        double* fi = a.Fim + grow;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const double ud = (double)y[i], kd = (double)kv[i];
            fr[i] = fma(a.fa_re, ud, fma(a.fb_re, kd, fr[i]));
            fi[i] = fma(a.fa_im, ud, fma(a.fb_im, kd, fi[i]));
        }
#pragma unroll 1
        for (int h = 1; h < args.nharm; ++h) {  // each harmonic filtered at its own frequency
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
// A whole period in one launch (PeriodArgs in launch.h): every workgroup keeps
// its 21 triangles resident -- state, stage combination and low parts in
// registers, stage input, geometry and matrices in LDS -- and the stages run
// in a loop, so no stage pays a launch or reads its state back.  The traces
// of edges between workgroups go through mailboxes of (value, epoch) pairs
// (tagged.h): after its update a workgroup writes its traces into its
// neighbours' mailboxes, and polls its own, which lie next to each other,
// until they carry the stage's epoch.  Two buffers alternate between epochs; a
// workgroup overwrites an epoch's mailbox two stages later, after it has read
// that neighbour's next epoch, which the neighbour wrote after reading this
// one.
//
// Four waves share a block: lanes own rows (triangle, component) as in
// k_stage2d, each wave a quarter of the nodes for the volume, lift and update
// work, and the threads together the 63 (q + 1) edge nodes of the flux, one
// each.  What bounds it: one stage is one exchange (0.4-0.6 us between a store
// and the poll that sees it) and one wave's chain of LDS round trips and
// arithmetic (a wave alone on its SIMD issues one VALU instruction in about 8
// clocks, so a single-wave form took twice as long).  Whole solves, per stage:
// 22500 triangles P3 FP32 9.2 us by stage launches, 3.8 here; 4096 triangles P1
// FP64 4.9 and 2.2; 20 members of 3600 triangles P3 FP32 22.3 and 13.6.
// Publishing whole rows and gathering them lane by lane took 42 us a stage at
// 22500 triangles: requests, not bytes, are what the exchange pays for.  The
// arithmetic is that of k_stage2d, term by term, so results agree bit for bit.
template <typename T, int Q>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 5 : 3, 8)))
void k_period2d(PeriodArgs a, int64_t per) {
    constexpr int NP = Dim2<Q>::NP, NFP = Dim2<Q>::NFP, NF3 = 3 * NFP;
    constexpr bool COMP = std::is_same<T, float>::value;
    using X = Tagged<T>;
    constexpr int W = 4, NTH = 64 * W, ROWS = EPB * 3;
    constexpr int NW = (NP + W - 1) / W;                     // nodes of a row per wave
    constexpr int GD = (2 * NW + 3) / 4, GL = (NW + 3) / 4;  // groups of four output rows (D_1 and D_2; LIFT)
    static_assert(ROWS * NFP <= NTH, "one flux node per thread");
    // rows in LDS, padded to whole 16-byte groups: stage input and D [.][DR],
    // flux [row][FR], LIFT [NP][FR]
    constexpr int PV = 16 / (int)sizeof(T);
    constexpr int DR = (NP + PV - 1) / PV * PV, FR = (NF3 + PV - 1) / PV * PV;
    constexpr int TO = ROWS * DR;      // received traces, then the flux, behind the staged block
    typedef T VM __attribute__((ext_vector_type(PV)));
    // stage input [row][DR]; traces [edge][component][edge node], replaced by the flux [row][FR]
    __shared__ __align__(16) T sS[TO + ROWS * FR];
    __shared__ __align__(16) T sD[COMP ? 1 : 2 * NP * DR];  // FP32: in registers
    __shared__ __align__(16) T sL[COMP ? 1 : NP * FR];
    __shared__ T sG[EPB * kGeo2];
    __shared__ int sX[ROWS];          // mailbox j: its edge, and the neighbour's mailbox
    __shared__ uint8_t sE[ROWS];
    __shared__ int sStop;

    const int mem = a.order ? a.order[a.first + blockIdx.y] : 0;
    const int64_t bx = blockIdx.x;
    const int64_t blk = (bx & 7) * per + (bx >> 3);  // consecutive blocks on one XCD
    const int64_t e0 = blk * EPB;
    if (e0 >= a.K) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ne = (int)((a.K - e0) < EPB ? (a.K - e0) : EPB);
    const int M = a.msteps ? a.msteps[mem] : a.M;
    const int S = a.scheme == 2 ? 2 : 4;
    const int el = lane / 3;
    const int c = lane - 3 * el;
    const bool act = el < ne;
    const int elc = act ? el : 0;
    const int row = elc * 3 + c;
    const int base = 3 * elc;
    const int i0 = wave * NW;  // this wave's nodes i0 .. i0 + NW - 1 (those below NP)
    const int64_t fo = (int64_t)mem * a.bstride;
    const int64_t grow = fo + (e0 * 3 + row) * NP + i0;
    const int x0 = a.xstart[blk];
    const int nitem = (a.xstart[blk + 1] - x0) * NF3;
    const T* gm = mats2<T>() + mat2_off(Q);
    // FP32: the wave's matrix rows as broadcast operands (mfma_rows), D's
    // rows being D_1 at the wave's nodes, then D_2
    float mD[(NP * GD + 15) / 16], mL[(NF3 * GL + 15) / 16];
    if constexpr (COMP) {
        mfma_operand<NP, GD>(mD, lane, [&](int rr, int k) {
            const int d = rr / NW, i = i0 + rr % NW;
            return d < 2 && i < NP ? (float)gm[(d * NP + i) * NP + k] : 0.f;
        });
        mfma_operand<NF3, GL>(mL, lane, [&](int u, int k) {
            return u < NW && i0 + u < NP ? (float)gm[2 * NP * NP + (i0 + u) * NF3 + k] : 0.f;
        });
    }
    {
        const T* geo = (const T*)a.geo + (int64_t)mem * a.gstride + e0 * kGeo2;
        for (int i = tid; i < ne * kGeo2; i += NTH) sG[i] = geo[i];
        if constexpr (!COMP) {
            for (int i = tid; i < 2 * NP * DR; i += NTH) sD[i] = i % DR < NP ? gm[i / DR * NP + i % DR] : T(0);
            for (int i = tid; i < NP * FR; i += NTH)
                sL[i] = i % FR < NF3 ? gm[2 * NP * NP + i / FR * NF3 + i % FR] : T(0);
        }
        for (int i = tid; i < TO + ROWS * FR; i += NTH) sS[i] = T(0);
        if (tid == 0) sStop = 0;
        if (tid < ne * 3) {
            const int id = a.xslot[e0 * 3 + tid];
            const int cd = a.conn[e0 * 3 + tid];
            if (id >= 0) {
                sE[id - x0] = (uint8_t)tid;
                sX[id - x0] = a.xslot[(int64_t)(cd >> 5) * 3 + ((cd >> 3) & 3)];
            }
        }
    }
    // own state: nodes i0 + u of the lane's row
    T up[NW], yo[NW], ap[NW];
    float lo[COMP ? NW : 1];
    bool mine[NW];
#pragma unroll
    for (int u = 0; u < NW; ++u) {
        mine[u] = act && i0 + u < NP;
        up[u] = mine[u] ? ((const T*)a.U)[grow + u] : T(0);
        yo[u] = up[u];
        ap[u] = T(0);
        if constexpr (COMP) lo[u] = mine[u] ? from_bf16(((const uint16_t*)a.Ulo)[grow + u]) : 0.f;
    }
    __syncthreads();

    // this thread's flux node, node k of edge t: LDS offsets of the own trace
    // and of the neighbour's (in the staged block, or received; a boundary's:
    // the own), packed; the place of the edge's geometry (12 bits) and of the
    // flux (12 bits) with what the neighbour is (8 bits): the offset between
    // its components, 0 on a wall with the PEC ghost, 1 with the impedance ghost
    static_assert(TO + ROWS * FR < 65536 && EPB * kGeo2 < 4096 && ROWS * FR < 4096 && NFP > 1 && DR < 256,
                  "packed offsets");
    uint32_t trace, place;
    {
        const int t = tid < ROWS * NFP ? tid / NFP : 0, k = tid < ROWS * NFP ? tid % NFP : 0;
        const int e = t / 3, f = t - 3 * e;
        const int code = t < ne * 3 ? a.conn[e0 * 3 + t] : -2;
        const int64_t nb = code >> 5;
        const int nf = (code >> 3) & 3, kk = (code & 7) ? NFP - 1 - k : k;
        const bool in = nb >= e0 && nb < e0 + ne;
        const int own = e * 3 * DR + edge_node<Q>(f, k);
        const int nbo = code < 0 ? own : in ? (int)(nb - e0) * 3 * DR + edge_node<Q>(nf, kk) : TO + t * NF3 + kk;
        const int what = code == -1 ? 0 : code < 0 ? 1 : in ? DR : NFP;
        trace = (uint32_t)own | ((uint32_t)nbo << 16);
        place = (uint32_t)(e * kGeo2 + 4 + 6 * f) | ((uint32_t)(e * 3 * FR + f * NFP + k) << 12) |
                ((uint32_t)what << 24);
    }
    // mailbox value i: its LDS source, its place with the neighbour, and where
    // the value received in its stead goes; a thread's first one is kept packed
    auto mail = [&](int i, int& src, uint32_t& dst, int& rcv) {
        const int j = i / NF3, r = i - j * NF3;
        const int cc = r / NFP, k = r - cc * NFP;
        const int t = sE[j], f = t % 3;
        src = (t - f + cc) * DR + edge_node<Q>(f, k);
        dst = (uint32_t)(sX[j] * NF3 + r) * X::W;
        rcv = TO + t * NF3 + r;
    };
    uint32_t mlds = 0, mdst = 0;
    if (tid < nitem) {
        int src, rcv;
        mail(tid, src, mdst, rcv);
        mlds = (uint32_t)src | ((uint32_t)rcv << 16);
    }

    uint32_t epoch = a.epoch;
    const int64_t half = (int64_t)a.members * a.next * (NF3 * X::W);  // words of one buffer
    unsigned long long* const xch = a.xch + (int64_t)mem * a.next * (NF3 * X::W);
    const unsigned long long* const inbox = xch + (int64_t)x0 * (NF3 * X::W);
    auto publish = [&]() {  // the stage input for this epoch, to LDS and to the neighbours
#pragma unroll
        for (int u = 0; u < NW; ++u)
            if (mine[u]) sS[row * DR + i0 + u] = yo[u];
        __syncthreads();
        unsigned long long* const q = xch + (epoch & 1) * half;
        if (tid < nitem) X::put(q + mdst, sS[mlds & 0xffffu], epoch);
        for (int i = tid + NTH; i < nitem; i += NTH) {
            int src, rcv;
            uint32_t dst;
            mail(i, src, dst, rcv);
            X::put(q + dst, sS[src], epoch);
        }
    };
    publish();

    const int srcA = c == 0 ? base + 2 : base;
    const int srcB = c == 0 ? base + 1 : base;
    const T sa = c == 1 ? T(0) : T(-1);
    const T sb = c == 2 ? T(0) : T(1);
    const bool src = c < a.src_rows;
    // RK4 with the filter ends with one more right-hand side at the last level
    const bool tail = a.filter && S == 4;
    for (int m = 0; m < M + (tail ? 1 : 0); ++m) {
        const int ns = m < M ? S : 1;
        for (int s = 0; s < ns; ++s) {
            // an offset of zero that the compiler cannot see: matrices and
            // geometry are read from LDS in every stage (hoisted out of the
            // loop they would take every register), and packed words are
            // unpacked there
            int z = 0;
            asm volatile("" : "+v"(z));
            asm volatile("" : "+v"(trace), "+v"(place), "+v"(mlds), "+v"(mdst));
            const double* tab = a.mtab + (((int64_t)(m < M ? m : a.M) * S + s) * a.members + mem) * kMemberParams;
            const T cy = (T)tab[0], ca = (T)tab[1], cu = (T)tab[2], scos = (T)tab[3], ssin = (T)tab[4];
            // request the neighbours' traces; they travel during the volume work
            const unsigned long long* const in = inbox + (epoch & 1) * half;
            Inbox<T, 1, NTH> box;
            box.request(in, 0, nitem, tid);

            // ---- volume: physical derivatives of the lane's component at the
            // wave's nodes, exchanged between the triangle's lanes
            const T* gg = &sG[elc * kGeo2 + z];
            T acc[NW];
            {
                T y[DR], r0[NW], r1[NW];
                const T* yr = &sS[row * DR + z];
                const T g00 = gg[0], g01 = gg[1], g10 = gg[2], g11 = gg[3];
#pragma unroll
                for (int v = 0; v < DR / PV; ++v) {
                    const VM t = *reinterpret_cast<const VM*>(yr + v * PV);
#pragma unroll
                    for (int u = 0; u < PV; ++u) y[v * PV + u] = t[u];
                }
                if constexpr (COMP) {
                    f32x4 d[GD] = {};
                    mfma_rows<NP, GD>(mD, y, d);
#pragma unroll
                    for (int u = 0; u < NW; ++u) {
                        r0[u] = d[u / 4][u % 4];
                        r1[u] = d[(NW + u) / 4][(NW + u) % 4];
                    }
                } else {
                    int zr[2] = {z, z};
#pragma unroll
                    for (int u = 0; u < NW; ++u) {
                        const int i = i0 + u < NP ? i0 + u : NP - 1;
                        const T* D = sD + zr[u & 1];
                        r0[u] = r1[u] = T(0);
#pragma unroll
                        for (int v = 0; v < DR / PV; ++v) {
                            const VM m0 = *reinterpret_cast<const VM*>(D + i * DR + v * PV);
                            const VM m1 = *reinterpret_cast<const VM*>(D + (NP + i) * DR + v * PV);
#pragma unroll
                            for (int w = 0; w < PV; ++w)
                                if (v * PV + w < NP) {
                                    r0[u] = fma(m0[w], y[v * PV + w], r0[u]);
                                    r1[u] = fma(m1[w], y[v * PV + w], r1[u]);
                                }
                        }
                        // the matrix rows of u + 2 are requested when u is done:
                        // all of them at once would take every register
                        asm volatile("" : "+v"(zr[u & 1]) : "v"(r1[u]));
                    }
                }
#pragma unroll
                for (int u = 0; u < NW; ++u) {
                    const T d1 = fma(g00, r0[u], g10 * r1[u]);
                    const T d2 = fma(g01, r0[u], g11 * r1[u]);
                    const T A = __shfl(d1, srcA);
                    const T B = __shfl(d2, srcB);
                    acc[u] = fma(sa, A, sb * B);
                }
            }

            if (!box.settle(in, nitem, tid, epoch, a, [&](int i, int r, T v) {
                    int src, rcv = (int)(mlds >> 16);
                    uint32_t dst;
                    if (r > 0) mail(i, src, dst, rcv);
                    sS[rcv] = v;
                }))
                sStop = 1;
            __syncthreads();
            if (sStop) return;

            // ---- upwind flux, all three components at the thread's edge node
            T fx[3];
            {
                const T* g = &sG[(place & 4095u) + z];
                const T* om = &sS[trace & 0xffffu];
                const T* np = &sS[trace >> 16];
                const int what = place >> 24;
                const int st = what > 1 ? what : DR;
                const T em = om[0], h1m = om[DR], h2m = om[2 * DR];
                T ep = np[0], h1p = np[st], h2p = np[2 * st];
                if (what == 0) ep = -em;  // PEC ghost: e+ = -e-, h+ = h-
                if (what == 1) ep = h1p = h2p = T(0);  // impedance ghost (homogeneous part): zero exterior state
                upwind2d(g, em, h1m, h2m, ep, h1p, h2p, fx);
            }
            __syncthreads();  // every trace is read
            if (tid < ROWS * NFP) {
                T* o = &sS[TO + ((place >> 12) & 4095u)];
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) o[cc * FR] = fx[cc];
            }
            __syncthreads();

            // ---- lift and update of the wave's nodes
            {
                T fl[FR];
                const T* fr = &sS[TO + row * FR];
#pragma unroll
                for (int v = 0; v < FR / PV; ++v) {
                    const VM t = *reinterpret_cast<const VM*>(fr + v * PV);
#pragma unroll
                    for (int w = 0; w < PV; ++w) fl[v * PV + w] = t[w];
                }
                if constexpr (COMP) {
                    f32x4 d[GL] = {};
#pragma unroll
                    for (int u = 0; u < NW; ++u) d[u / 4][u % 4] = acc[u];
                    mfma_rows<NF3, GL>(mL, fl, d);
#pragma unroll
                    for (int u = 0; u < NW; ++u) acc[u] = d[u / 4][u % 4];
                } else {
                    int zr[2] = {z, z};
#pragma unroll
                    for (int u = 0; u < NW; ++u) {
                        const int i = i0 + u < NP ? i0 + u : NP - 1;
                        const T* L = sL + zr[u & 1];
#pragma unroll
                        for (int v = 0; v < FR / PV; ++v) {
                            const VM t = *reinterpret_cast<const VM*>(L + i * FR + v * PV);
#pragma unroll
                            for (int w = 0; w < PV; ++w)
                                if (v * PV + w < NF3) acc[u] = fma(t[w], fl[v * PV + w], acc[u]);
                        }
                        asm volatile("" : "+v"(zr[u & 1]) : "v"(acc[u]));
                    }
                }
            }
            const T inv = gg[c == 0 ? 22 : 23];
            const T sig = c == 0 ? gg[24] : T(0);
            T kv[NW];
#pragma unroll
            for (int u = 0; u < NW; ++u) kv[u] = fma(inv, acc[u], -sig * yo[u]);
            if (src) {
                const int64_t so = (int64_t)mem * a.sstride + (e0 * 3 + row) * NP + i0;
#pragma unroll
                for (int u = 0; u < NW; ++u)
                    if (mine[u])
                        kv[u] = fma(scos, ((const T*)a.Sre)[so + u], fma(-ssin, ((const T*)a.Sim)[so + u], kv[u]));
            }
            if (a.filter && s == 0) {
                const double fa_re = tab[5], fa_im = tab[6], fb_re = tab[7], fb_im = tab[8];
                double* fr = a.Fre + grow;
                double* fi = a.Fim + grow;
#pragma unroll
                for (int u = 0; u < NW; ++u)
                    if (mine[u]) {
                        const double ud = (double)yo[u], kd = (double)kv[u];
                        fr[u] = fma(fa_re, ud, fma(fb_re, kd, fr[u]));
                        fi[u] = fma(fa_im, ud, fma(fb_im, kd, fi[u]));
                    }
            }
            if (m >= M) break;  // the last level's right-hand side: filter only
            const bool last = s == S - 1;
            if (!last) {
#pragma unroll
                for (int u = 0; u < NW; ++u) {
                    if (S == 4) ap[u] = s > 0 ? fma(ca, kv[u], ap[u]) : COMP ? ca * kv[u] : fma(ca, kv[u], yo[u]);
                    yo[u] = fma(cy, kv[u], up[u]);
                }
            } else {
#pragma unroll
                for (int u = 0; u < NW; ++u) {
                    if constexpr (COMP) {
                        float sum, e;
                        two_sum(up[u], S == 4 ? fma(cu, kv[u], ap[u]) + lo[u] : fma(cu, kv[u], lo[u]), sum, e);
                        up[u] = sum;
                        lo[u] = from_bf16(to_bf16(e));
                    } else {
                        up[u] = fma(cu, kv[u], S == 4 ? ap[u] : up[u]);
                    }
                    yo[u] = up[u];
                }
            }
            if (m + 1 < M || !last || tail) {
                ++epoch;
                publish();
            }
        }
    }
#pragma unroll
    for (int u = 0; u < NW; ++u)
        if (mine[u]) {
            ((T*)a.U)[grow + u] = up[u];
            if constexpr (COMP) ((uint16_t*)a.Ulo)[grow + u] = to_bf16(lo[u]);
        }
}

template <typename T>
__global__ void k_to_field2d(const double* __restrict__ X, T* __restrict__ U, uint16_t* __restrict__ Ulo, int64_t n,
                             int Np, int flipH) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double x = X[i];
        if (flipH && ((i / Np) % 3) >= 1) x = -x;
        const T hi = (T)x;
        U[i] = hi;
        if constexpr (std::is_same<T, float>::value)
            if (Ulo) Ulo[i] = to_bf16((float)(x - (double)hi));
    }
}

template <typename T>
__global__ void k_from_field2d(const T* __restrict__ U, const uint16_t* __restrict__ Ulo, double* __restrict__ Yo,
                               const double* __restrict__ sub, int64_t n, int Np, int flipH) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double x = (double)U[i];
        if constexpr (std::is_same<T, float>::value)
            if (Ulo) x += (double)from_bf16(Ulo[i]);
        if (flipH && ((i / Np) % 3) >= 1) x = -x;
        if (sub) x -= sub[i];
        Yo[i] = x;
    }
}

constexpr int kDot2Blocks = 1024;
constexpr int kDot2Threads = 256;

// (U, V)_{eps,mu} per block over rows r = 3 e + c (weight wE for c = 0, wH
// otherwise), fixed decomposition; k_dot2d_final sums the partials in a
// fixed order, so the result does not depend on scheduling.
template <int Q>
__global__ __launch_bounds__(kDot2Threads) void k_dot2d(const double* __restrict__ U, const double* __restrict__ V,
                                                        const double* __restrict__ wE, const double* __restrict__ wH,
                                                        int64_t K, double* __restrict__ partial) {
    constexpr int NP = Dim2<Q>::NP;
    constexpr int MMO = mat2_off(Q) + 2 * NP * NP + NP * 3 * Dim2<Q>::NFP;
    __shared__ double sm[kDot2Threads];
    double acc = 0.0;
    const int64_t rows = 3 * K;
    for (int64_t r = blockIdx.x * (int64_t)kDot2Threads + threadIdx.x; r < rows;
         r += (int64_t)gridDim.x * kDot2Threads) {
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
            for (int j = 0; j < NP; ++j) mvv = fma(c2Mat64[MMO + i * NP + j], vv[j], mvv);
            s = fma(u[i], mvv, s);
        }
        const int64_t e = r / 3;
        acc = fma(s, (r - 3 * e) == 0 ? wE[e] : wH[e], acc);
    }
    sm[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kDot2Threads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sm[threadIdx.x] += sm[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sm[0];
}

// Batched form: member b = blockIdx.y, the same block decomposition and
// summation order per member (a member's inner product equals its single one).
template <int Q>
__global__ __launch_bounds__(kDot2Threads) void k_dot2d_batch(const double* __restrict__ U,
                                                              const double* __restrict__ V,
                                                              const double* __restrict__ wE,
                                                              const double* __restrict__ wH, int64_t wstride,
                                                              int64_t K, double* __restrict__ partial) {
    constexpr int NP = Dim2<Q>::NP;
    constexpr int MMO = mat2_off(Q) + 2 * NP * NP + NP * 3 * Dim2<Q>::NFP;
    __shared__ double sm[kDot2Threads];
    const int64_t bm = blockIdx.y;
    const int64_t n = 3 * K * NP;
    U += bm * n;
    V += bm * n;
    wE += bm * wstride;
    wH += bm * wstride;
    double acc = 0.0;
    const int64_t rows = 3 * K;
    for (int64_t r = blockIdx.x * (int64_t)kDot2Threads + threadIdx.x; r < rows;
         r += (int64_t)gridDim.x * kDot2Threads) {
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
            for (int j = 0; j < NP; ++j) mvv = fma(c2Mat64[MMO + i * NP + j], vv[j], mvv);
            s = fma(u[i], mvv, s);
        }
        const int64_t e = r / 3;
        acc = fma(s, (r - 3 * e) == 0 ? wE[e] : wH[e], acc);
    }
    sm[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kDot2Threads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sm[threadIdx.x] += sm[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[bm * kDot2Blocks + blockIdx.x] = sm[0];
}

__global__ __launch_bounds__(kDot2Threads) void k_dot2d_final_batch(const double* __restrict__ partial, int n,
                                                                    double* __restrict__ out) {
    __shared__ double sm[kDot2Threads];
    const int bm = blockIdx.x;
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += kDot2Threads) acc += partial[(int64_t)bm * kDot2Blocks + i];
    sm[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kDot2Threads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sm[threadIdx.x] += sm[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[bm] = sm[0];
}

__global__ __launch_bounds__(kDot2Threads) void k_dot2d_final(const double* __restrict__ partial, int n,
                                                              double* __restrict__ out) {
    __shared__ double sm[kDot2Threads];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += kDot2Threads) acc += partial[i];
    sm[threadIdx.x] = acc;
    __syncthreads();
    for (int s = kDot2Threads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sm[threadIdx.x] += sm[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = sm[0];
}

unsigned grid2_for(int64_t n) {
    int64_t g = (n + 255) / 256;
    if (g > 4096) g = 4096;
    if (g < 1) g = 1;
    return (unsigned)g;
}

void check2() {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) fail(CMCG_ERR_DEVICE, std::string("2-D kernel launch: ") + hipGetErrorString(e));
}

template <typename T, int Q>
void stage2d(const StageArgs& a, hipStream_t s) {
    const int64_t nb = (a.K + EPB - 1) / EPB;
    const int64_t per = (nb + 7) / 8;
    if (8 * per > 0x7fffffffLL) fail(CMCG_ERR_ARG, "stage2d: too many element blocks");
    if (a.mtab && (a.nmembers < 1 || a.nmembers > 65535)) fail(CMCG_ERR_ARG, "stage2d: 1 to 65535 members");
    const dim3 grid((unsigned)(8 * per), (unsigned)(a.mtab ? a.nmembers : 1));
    // early loads pay off while the launch has at most about two single-wave
    // workgroups per SIMD (1024 SIMDs); FP64 always takes the lean form
    const int64_t total = nb * (a.mtab ? a.nmembers : 1);
    if constexpr (std::is_same<T, float>::value) {
        if (total <= kEarlyBlocks) {
            hipLaunchKernelGGL((k_stage2d<T, Q, true>), grid, dim3(64), 0, s, a, per);
            return;
        }
    }
    hipLaunchKernelGGL((k_stage2d<T, Q, false>), grid, dim3(64), 0, s, a, per);
}

template <typename F> auto period2d_kernel(int q, int precision, F f) {
    if (precision == CMCG_FP64) {
        if (q == 1) return f(k_period2d<double, 1>);
        return q == 2 ? f(k_period2d<double, 2>) : f(k_period2d<double, 3>);
    }
    if (q == 1) return f(k_period2d<float, 1>);
    return q == 2 ? f(k_period2d<float, 2>) : f(k_period2d<float, 3>);
}

}  // namespace

void upload_constants2d(int q, const double* D, const double* LIFT, const double* M, const int* fnode) {
    const int NP = np2_of(q), NFP = nfp2_of(q);
    for (int f = 0; f < 3; ++f)
        for (int k = 0; k < NFP; ++k) {
            const int want = q == 1 ? edge_node<1>(f, k) : q == 2 ? edge_node<2>(f, k) : edge_node<3>(f, k);
            if (fnode[f * NFP + k] != want) fail(CMCG_ERR_ARG, "2-D edge-node table does not match the kernels");
        }
    const int n = 2 * NP * NP + NP * 3 * NFP + NP * NP;
    std::vector<double> buf(n);
    std::copy(D, D + 2 * NP * NP, buf.begin());
    std::copy(LIFT, LIFT + NP * 3 * NFP, buf.begin() + 2 * NP * NP);
    std::copy(M, M + NP * NP, buf.begin() + 2 * NP * NP + 3 * NP * NFP);
    std::vector<float> bf(buf.begin(), buf.end());
    const size_t off = mat2_off(q);
    CMCG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c2Mat64), buf.data(), n * sizeof(double), off * sizeof(double),
                               hipMemcpyHostToDevice));
    CMCG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c2Mat32), bf.data(), n * sizeof(float), off * sizeof(float),
                               hipMemcpyHostToDevice));
}

void launch_stage2d(int q, int precision, const StageArgs& a, hipStream_t s) {
    if (precision == CMCG_FP64) {
        if (q == 1) stage2d<double, 1>(a, s);
        else if (q == 2) stage2d<double, 2>(a, s);
        else stage2d<double, 3>(a, s);
    } else {
        if (q == 1) stage2d<float, 1>(a, s);
        else if (q == 2) stage2d<float, 2>(a, s);
        else stage2d<float, 3>(a, s);
    }
    check2();
}

int64_t period_room2d(int q, int precision) {
    return period2d_kernel(q, precision, [](auto kernel) { return resident_room(kernel, 256); });
}

void launch_period2d(int q, int precision, const PeriodArgs& a, int n, int left_out, hipStream_t s) {
    period2d_kernel(q, precision, [&](auto kernel) {
        launch_resident(kernel, (a.K + EPB - 1) / EPB, n, left_out, 256, a, s);
    });
}

void launch_to_field2d(int precision, int Np, const double* X, void* U, void* Ulo, int64_t n, int flipH,
                       hipStream_t s) {
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_to_field2d<double>, dim3(grid2_for(n)), dim3(256), 0, s, X, (double*)U, nullptr, n, Np,
                           flipH);
    else
        hipLaunchKernelGGL(k_to_field2d<float>, dim3(grid2_for(n)), dim3(256), 0, s, X, (float*)U, (uint16_t*)Ulo, n,
                           Np, flipH);
    check2();
}

void launch_from_field2d(int precision, int Np, const void* U, const void* Ulo, double* Y, const double* sub,
                         int64_t n, int flipH, hipStream_t s) {
    if (precision == CMCG_FP64)
        hipLaunchKernelGGL(k_from_field2d<double>, dim3(grid2_for(n)), dim3(256), 0, s, (const double*)U, nullptr, Y,
                           sub, n, Np, flipH);
    else
        hipLaunchKernelGGL(k_from_field2d<float>, dim3(grid2_for(n)), dim3(256), 0, s, (const float*)U,
                           (const uint16_t*)Ulo, Y, sub, n, Np, flipH);
    check2();
}

void launch_dot_batch2d(int q, const double* U, const double* V, const double* wE, const double* wH,
                        int64_t wstride, int64_t K, int B, double* partial, double* out_dev, hipStream_t s) {
    const dim3 grid(kDot2Blocks, (unsigned)B);
    if (q == 1)
        hipLaunchKernelGGL(k_dot2d_batch<1>, grid, dim3(kDot2Threads), 0, s, U, V, wE, wH, wstride, K, partial);
    else if (q == 2)
        hipLaunchKernelGGL(k_dot2d_batch<2>, grid, dim3(kDot2Threads), 0, s, U, V, wE, wH, wstride, K, partial);
    else
        hipLaunchKernelGGL(k_dot2d_batch<3>, grid, dim3(kDot2Threads), 0, s, U, V, wE, wH, wstride, K, partial);
    hipLaunchKernelGGL(k_dot2d_final_batch, dim3((unsigned)B), dim3(kDot2Threads), 0, s, partial, kDot2Blocks,
                       out_dev);
    check2();
}

int dot2d_partials() { return kDot2Blocks; }

void launch_dot2d(int q, const double* U, const double* V, const double* wE, const double* wH, int64_t K,
                  double* partial, double* out_dev, hipStream_t s) {
    if (q == 1)
        hipLaunchKernelGGL(k_dot2d<1>, dim3(kDot2Blocks), dim3(kDot2Threads), 0, s, U, V, wE, wH, K, partial);
    else if (q == 2)
        hipLaunchKernelGGL(k_dot2d<2>, dim3(kDot2Blocks), dim3(kDot2Threads), 0, s, U, V, wE, wH, K, partial);
    else
        hipLaunchKernelGGL(k_dot2d<3>, dim3(kDot2Blocks), dim3(kDot2Threads), 0, s, U, V, wE, wH, K, partial);
    hipLaunchKernelGGL(k_dot2d_final, dim3(1), dim3(kDot2Threads), 0, s, partial, kDot2Blocks, out_dev);
    check2();
}

}  // namespace cmcg
