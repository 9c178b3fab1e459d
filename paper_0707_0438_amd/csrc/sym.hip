// Pairwise sums of one self-gravitating set in which every pair of particles
// is evaluated once and serves both of its particles (double-single
// arithmetic, eps > 0).
//
// The general kernel (force.hip) evaluates each pair twice, once for either
// particle: 34 VALU instructions an interaction, and it runs at the VALU
// issue limit.  What depends on the pair alone (relative position and
// velocity, r^-1, r.u, alpha, u - alpha r) takes 25 of them, so a pair that
// serves both sides takes 25 + 2 x 9 = 43, or 21.5 an interaction.
//
// Layout.  A wave holds 256 consecutive i-particles, four to a lane (lane p:
// 4p .. 4p + 3), with their sums in registers.  j-particles stream through
// the lanes: at step t lane p meets j = t - p, reads its record from LDS and
// adds to two sets of sums: those of its own four i (registers), and those
// of j, which move with j from lane to lane (seven DPP moves a step,
// shared by four pairs).  A chain of ROW lanes thus hands j past 4 ROW
// consecutive i in ascending order, and an i meets j in ascending order, so
// both float32 partial sums run over exactly the 4 ROW = TJ consecutive
// partners, in the order, that a j-tile of the general kernel has: the
// partial sums are the general kernel's bit for bit, and only the sums over
// tiles (a two-sum there, float64 here) are formed in another order.  ROW =
// 16 (a DPP row, four chains a wave) or 64 lanes gives TJ = 64 or 256.
//
// The skew costs ROW steps per stream to fill.  Lane p reaches the end of a
// j-tile p steps after lane 0; there it parks its 28 partial sums in LDS
// and starts from zero, and whenever 16 lanes have done so the wave adds them
// to their float64 rows, a lane taking one i.
//
// What bounds it: VALU issue, at a clock that follows the power (2.08 GHz
// measured).  Seven DPP moves and four v_rsq a step issue at less than the
// full rate, so they stand together, with the LDS traffic, at raised priority
// (see rsq_group): 36.0 ms with them spread through the step, 32.6 as a
// group, 31.1 with the priority (2^18 bodies).  128 registers, four waves per
// SIMD; the sums over tiles live in memory as float64, which costs one
// read-add-write of 28 values a lane and tile.  The step is 181 VALU
// instructions for 8 interactions, 22.6 against the general kernel's 34.8.
// Measured, general kernel to this: 2^20 bodies 652 to 499 ms, 2^18 41.8 to
// 31 ms, 40000 1.20 to 1.02 ms; force only, 2^17 7.3 to 5.0 ms.
//
// Work.  The set is cut into nb blocks of lb particles (the last one padded)
// that stand in a ring.  Block A meets itself (one-sided, the self pair
// masked) and the blocks A + 1 .. A + nb / 2 after it (for nb even, one less
// from A = nb / 2 on), so every two blocks meet once: a contiguous stretch of
// the ring, cut into pieces of equal length.  A work item is one block's i
// against one piece of its stretch; a work-group of four waves takes 1024 i
// at a time.  Each piece owns a float64 row of sums for i and each block
// distance one for j, which the reduction adds in a fixed order.
#include "nbody_internal.h"

namespace nb {

constexpr float kSymPad = 1.0e18f;   // far-away position of padding records

// Value of the lane before; the first lane (of a 16-lane row, ROW = 16; else
// of the wave) gets 0.
template <int ROW>
__device__ __forceinline__ float sym_hop(float v) {
    constexpr int kCtrl = ROW == 16 ? 0x111 /* row_shr:1 */ : 0x138 /* wave_shr:1 */;
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, true));
}

// The lanes of `mask` store v at LDS byte offset `at`: no branch, so the
// step stays one basic block that the compiler can schedule as a whole.
template <int OFF>
__device__ __forceinline__ void sym_lds_store(uint64_t mask, uint32_t at, float4 v) {
    uint64_t keep;
    typedef float vec4 __attribute__((ext_vector_type(4)));
    const vec4 w = {v.x, v.y, v.z, v.w};
    asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, %1\n\tds_write_b128 %2, %3 offset:%4\n\ts_mov_b64 exec, %0"
                 : "=&s"(keep)
                 : "s"(mask), "v"(at), "v"(w), "n"(OFF)
                 : "memory");
}

// End of block A's stretch in this band.
__device__ __forceinline__ int sym_end(const SymArgs& a, int A) {
    return a.half && A >= a.nb / 2 ? a.off1 - a.lb : a.off1;
}

// KIND 0: acceleration, jerk, potential; 1: acceleration, potential.
// Quantities in the order ax ay az pot jx jy jz.
template <int TJ, int KIND>
__global__ __launch_bounds__(256, 4) void sym_kernel(SymArgs a) {
    static_assert(TJ == 64 || TJ == 256, "chains of 16 or 64 lanes");
    constexpr int ROW = TJ / 4;
    constexpr int ROWS = 64 / ROW;
    constexpr int PH = ROW == 16 ? 32 : 64;         // steps between two barriers
    constexpr int SPAN = ROW + PH;                  // records the lanes read in a phase
    constexpr int NQ = KIND == 1 ? 4 : 7;
    constexpr int NX = KIND == 1 ? 1 : 2;           // float4 per exit
    // records {hi, m}, {v, lo z}, {lo x, lo y} of the ROW j before a phase
    // and its PH, for this phase and the next
    __shared__ float4 recs[2][2 * SPAN + 1];
    __shared__ float2 recs2[2 * SPAN + 1];
    __shared__ float4 exits[4][PH * ROWS][NX];      // sums of the j that left a chain
    // sums of 16 lanes' i that ended a j-tile, one row of 64 i a quantity
    __shared__ float4 parked[4][NQ][16];

    if (a.bad && *a.bad == a.epoch) return;   // i_self is not the identity: the general kernel runs
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int p = lane & (ROW - 1);
    const int A = blockIdx.x % a.nb, piece = blockIdx.x / a.nb;
    const int n = a.n, ns = a.ns, ring = a.nb * a.lb;
    // ring offsets o0 .. o1 from the start of block A
    const int o0 = a.off0 + piece * a.lp;
    const int o1 = min(o0 + a.lp, sym_end(a, A));
    if (o0 >= o1) return;

    float eps2;   // in a VGPR: an SGPR operand halves the issue rate
    asm volatile("v_mov_b32 %0, %1" : "=v"(eps2) : "s"(a.eps2));
    // lanes at the end of a chain
    constexpr uint64_t kLast = ROW == 16 ? 0x8000800080008000ull : 1ull << 63;

    // staging of one PH-record chunk by the first 3 PH threads
    const int sr = tid / 3, sc = tid - 3 * sr;
    const bool stager = tid < 3 * PH;
    auto fetch = [&](int off, int end) {   // records at ring offsets off .. off + PH - 1
        float4 r = sc == 0 ? make_float4(kSymPad, kSymPad, kSymPad, 0.f) : make_float4(0.f, 0.f, 0.f, 0.f);
        int j = A * a.lb + off;
        if (j >= ring) j -= ring;
        if (stager && off < end && j + sr < n) r = a.pack[(size_t)j * 3 + tid];
        return r;
    };
    auto stage = [&](int at, const float4& r) {
        if (!stager) return;
        if (sc == 0) recs[0][at] = r;
        else if (sc == 1) *(float3*)&recs[1][at] = make_float3(r.x, r.y, r.z);
        else {
            recs[1][at].w = r.z;
            recs2[at] = make_float2(r.x, r.y);
        }
    };
    const int groups = (a.lb + 1023) / 1024;
    for (int g = 0; g < groups; ++g) {
        const int gbase = A * a.lb + 1024 * g;
        if (gbase >= n) break;
        const int live = min(4, (n - gbase + 255) / 256);   // waves that hold particles
        const int i0 = gbase + 256 * wave + 4 * lane;
        float ix[4], iy[4], iz[4], lx[4], ly[4], lz[4], iu[4], iv[4], iw[4], mn[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            // beyond the set: massless, far from the padding records too
            float4 r0 = make_float4(-kSymPad, -kSymPad, -kSymPad, 0.f);
            float4 r1 = make_float4(0.f, 0.f, 0.f, 0.f), r2 = r1;
            if (i0 + k < n) {
                const float4* r = a.pack + (size_t)(i0 + k) * 3;
                r0 = r[0];
                if (KIND != 1) r1 = r[1];
                r2 = r[2];
            }
            ix[k] = r0.x; iy[k] = r0.y; iz[k] = r0.z; mn[k] = -r0.w;
            iu[k] = r1.x; iv[k] = r1.y; iw[k] = r1.z;
            lx[k] = r2.x; ly[k] = r2.y; lz[k] = r2.z;
            // keeps the minus sign in the register: folded into the products
            // it would turn the j side's fused multiply-adds into three-
            // operand forms
            asm volatile("" : "+v"(mn[k]));
        }
        float acc[4][NQ];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int q = 0; q < NQ; ++q) acc[k][q] = 0.f;
        float ja[NQ];   // sums of the j in this lane, of opposite sign to acc's (mn is negative)
#pragma unroll
        for (int q = 0; q < NQ; ++q) ja[q] = 0.f;

        // Four i against one j record, the mass of j in mj[k] for i slot k;
        // BOTH: j's sums too.  aside(): what else breaks the stream of
        // full-rate instructions.
        auto pairs = [&](auto both, const float4& q0, const float4& q1, const float2& q2, const float* mj, auto aside) {
            constexpr bool BOTH = decltype(both)::value;
            float dx[4], dy[4], dz[4], s[4], rinv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                dx[k] = (q0.x - ix[k]) + (q2.x - lx[k]);
                dy[k] = (q0.y - iy[k]) + (q2.y - ly[k]);
                dz[k] = (q0.z - iz[k]) + (q1.w - lz[k]);
                s[k] = fmaf(dz[k], dz[k], fmaf(dy[k], dy[k], fmaf(dx[k], dx[k], eps2)));
            }
            // the instructions that issue at less than the full rate, together
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(3);
            aside();
            if (BOTH) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) ja[q] = sym_hop<ROW>(ja[q]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) rinv[k] = __builtin_amdgcn_rsqf(s[k]);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float rinv2 = rinv[k] * rinv[k];
                float tx = 0.f, ty = 0.f, tz = 0.f;
                if (KIND != 1) {
                    const float ux = q1.x - iu[k], uy = q1.y - iv[k], uz = q1.z - iw[k];
                    const float rv = fmaf(dz[k], uz, fmaf(dy[k], uy, dx[k] * ux));
                    const float al = 3.0f * rv * rinv2;
                    tx = fmaf(-al, dx[k], ux);
                    ty = fmaf(-al, dy[k], uy);
                    tz = fmaf(-al, dz[k], uz);
                }
                auto add = [&](float* s, float m) {
                    const float w = (m * rinv[k]) * rinv2;
                    s[0] = fmaf(w, dx[k], s[0]);
                    s[1] = fmaf(w, dy[k], s[1]);
                    s[2] = fmaf(w, dz[k], s[2]);
                    s[3] = fmaf(m, rinv[k], s[3]);
                    if (KIND != 1) {
                        s[NQ - 3] = fmaf(w, tx, s[NQ - 3]);
                        s[NQ - 2] = fmaf(w, ty, s[NQ - 2]);
                        s[NQ - 1] = fmaf(w, tz, s[NQ - 1]);
                    }
                };
                add(acc[k], mj[k]);
                if (BOTH) add(ja, mn[k]);
            }
        };
        // Adds the float32 sums over one j-tile of 16 lanes' i (first lane
        // 16 u; ROW = 16: lanes 4 u .. 4 u + 3 of each row), parked in LDS,
        // to their float64 rows: a lane takes one i.
        bool fresh = true;
        auto flush = [&](int u) {
            const int k = ROW == 16 ? 64 * (lane >> 4) + 16 * u + (lane & 15) : 64 * u + lane;
            const int i = gbase + 256 * wave + k;
            __builtin_amdgcn_wave_barrier();   // the parked sums come from other lanes
            if (i >= n) return;
            double* o = a.own + (size_t)piece * NQ * ns + i;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const double v = (double)((const float*)parked[wave][q])[lane];
                o[(size_t)q * ns] = fresh ? v : o[(size_t)q * ns] + v;
            }
        };
        // Parks this lane's sums (of its four i) and starts from zero.
        auto park = [&]() {
            __builtin_amdgcn_wave_barrier();   // the lanes before have read theirs
            const int at = ROW == 16 ? 4 * (lane >> 4) + (lane & 3) : lane & 15;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                parked[wave][q][at] = make_float4(acc[0][q], acc[1][q], acc[2][q], acc[3][q]);
                acc[0][q] = acc[1][q] = acc[2][q] = acc[3][q] = 0.f;
            }
        };
        auto flush_all = [&]() {
            for (int u = 0; u < 4; ++u) {
                if ((ROW == 16 ? p >> 2 : lane >> 4) == u) park();
                flush(u);
            }
            fresh = false;
        };
        const std::integral_constant<bool, false> own{};
        const std::integral_constant<bool, true> both{};

        // the block itself
        const int e0 = min(o1, a.lb);
        for (int o = o0; o < e0; o += PH) {
            const float4 r = fetch(o, e0);
            __syncthreads();
            stage(sr, r);
            __syncthreads();
            const int js = A * a.lb + o - i0;   // own index of i slot k: record k - js
#pragma unroll 1
            for (int s = 0; s < PH; ++s) {
                const float4 q0 = recs[0][s], q1 = recs[1][s];
                const float2 q2 = recs2[s];
                float m[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) m[k] = s + js == k ? 0.f : q0.w;
                pairs(own, q0, q1, q2, m, [] {});
            }
            if ((o + PH) % TJ == 0) flush_all();
        }
        // the blocks after it
        const int u0 = max(o0, a.lb), nch = (o1 - u0) / PH;
        if (nch > 0) {
            float4 cur = fetch(u0, o1), nxt;
            __syncthreads();
            if (sr >= PH - ROW) stage(sr - (PH - ROW), fetch(o1, o1));   // padding
            stage(ROW + sr, cur);
            __syncthreads();
            for (int h = 0; h <= nch; ++h) {
                const int buf = (h & 1) * SPAN;
                nxt = fetch(u0 + PH * (h + 1), o1);
                if (wave < live) {
                    const float4* r0 = &recs[0][buf + ROW - p];
                    const float4* r1 = &recs[1][buf + ROW - p];
                    const float2* r2 = &recs2[buf + ROW - p];
                    uint32_t ex = (uint32_t)(uintptr_t)&exits[wave][lane / ROW][0];
                    float4 q0 = r0[0], q1 = r1[0];
                    float2 q2 = r2[0];
                    auto step = [&](auto cross, int s) {
                        if (decltype(cross)::value && p == s) park();   // the j-tile is done for this lane
                        float4 n0, n1;
                        float2 n2;
                        const float m[4] = {q0.w, q0.w, q0.w, q0.w};
                        pairs(both, q0, q1, q2, m, [&] {
                            // the j that the step before took to the end of its chain
                            sym_lds_store<0>(kLast, ex, make_float4(ja[0], ja[1], ja[2], ja[3]));
                            if (KIND != 1)
                                sym_lds_store<16>(kLast, ex, make_float4(ja[NQ - 3], ja[NQ - 2], ja[NQ - 1], 0.f));
                            ex += ROWS * NX * 16;
                            n0 = r0[s + 1];
                            n1 = r1[s + 1];
                            n2 = r2[s + 1];
                        });
                        q0 = n0;
                        q1 = n1;
                        q2 = n2;
                    };
                    const bool tile = h > 0 && h < nch && h % (TJ / PH) == 0;   // a j-tile ends in this phase
                    int s = 0;
                    if (tile) {
                        constexpr int W = ROW / 4 < 16 ? ROW / 4 : 16;   // steps in which 16 lanes end their tile
                        for (int u = 0; u < ROW / W; ++u) {
#pragma unroll 1
                            for (const int e = s + W; s < e; ++s) step(both, s);
                            flush(u);
                        }
                        fresh = false;
                    }
                    const int end = h < nch ? PH : ROW;
#pragma unroll 2
                    for (; s < end; s += 2) {
                        step(own, s);
                        step(own, s + 1);
                    }
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the exits' stores
                }
                if (sr >= PH - ROW) stage((SPAN - buf) + sr - (PH - ROW), cur);
                stage((SPAN - buf) + ROW + sr, nxt);
                cur = nxt;
                __syncthreads();
                // the j that left the chains in this phase: the sums of the
                // work-group's 1024 i
                for (int e = tid; e < PH * 4; e += 256) {
                    const int at = e & (PH - 1), q = e / PH;
                    const int off = u0 + PH * h + at - ROW;
                    if (off < u0 || off >= o1) continue;
                    int j = A * a.lb + off;
                    if (j >= ring) j -= ring;
                    if (j >= n) continue;
#pragma unroll
                    for (int x = 0; x < NX; ++x) {
                        if (x == 1 && q == 3) break;
                        double s = 0.0;
                        for (int w = 0; w < live; ++w)
#pragma unroll
                            for (int r = 0; r < ROWS; ++r)
                                s += (double)((const float*)&exits[w][at * ROWS + r][x])[q];
                        if (x == 0 && q == 3) s = -s;   // the potential does not turn its sign with r
                        double* o = a.partner + ((size_t)((off - a.off0) >> a.lbs) * NQ + 4 * x + q) * ns + j;
                        *o = g == 0 ? s : *o + s;
                    }
                }
                __syncthreads();
            }
            if (wave < live) flush_all();
        }
    }
}

// Sums of one band of distances, in a fixed order, added to the rows of the
// bands before; the last band applies G.
template <int NQ>
__global__ __launch_bounds__(256) void sym_reduce_kernel(SymArgs a) {
    if (a.bad && *a.bad == a.epoch) return;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)NQ * a.n) return;
    const int q = (int)(t / a.n);
    const int i = (int)(t - (int64_t)q * a.n);
    const int A = i >> a.lbs;
    double s = 0.0;
    const int np = (sym_end(a, A) - a.off0 + a.lp - 1) / a.lp;
    for (int k = 0; k < np; ++k) s += a.own[((size_t)k * NQ + q) * a.ns + i];
    for (int d = max(1, a.off0 >> a.lbs); d < a.off1 >> a.lbs; ++d) {
        const int from = A >= d ? A - d : A - d + a.nb;   // the block whose stretch holds i at distance d
        if (d << a.lbs >= sym_end(a, from)) continue;
        s += a.partner[((size_t)(d - (a.off0 >> a.lbs)) * NQ + q) * a.ns + i];
    }
    double* o = a.out[q] + i;
    if (!a.first) s += *o;
    if (a.last) s = q == 3 ? -a.G * s : a.G * s;
    *o = s;
}

hipError_t launch_sym(int tile_j, int kind, int items, const SymArgs& a, hipStream_t st) {
    const dim3 g(items), b(256);
    if (tile_j == 64 && kind == 0) hipLaunchKernelGGL((sym_kernel<64, 0>), g, b, 0, st, a);
    else if (tile_j == 64 && kind == 1) hipLaunchKernelGGL((sym_kernel<64, 1>), g, b, 0, st, a);
    else if (tile_j == 256 && kind == 0) hipLaunchKernelGGL((sym_kernel<256, 0>), g, b, 0, st, a);
    else if (tile_j == 256 && kind == 1) hipLaunchKernelGGL((sym_kernel<256, 1>), g, b, 0, st, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_sym_reduce(int kind, const SymArgs& a, hipStream_t st) {
    const int64_t t = (int64_t)(kind == 1 ? 4 : 7) * a.n;
    const dim3 g((unsigned)((t + 255) / 256)), b(256);
    if (kind == 1) hipLaunchKernelGGL(sym_reduce_kernel<4>, g, b, 0, st, a);
    else hipLaunchKernelGGL(sym_reduce_kernel<7>, g, b, 0, st, a);
    return hipGetLastError();
}

}  // namespace nb
