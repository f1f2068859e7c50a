// pairs.hip -- the per-layer adjoint gradient by the explicit pair formulation of
// Prop. 2 and Eq. "capped": every adjoint state
//     lambda^{t,i}[d,n] = g_t[d] C_t[n] prod_{j=i+1}^{t} a_j[d,n]
// for the pairs (t, i) of the window (i <= t < i + tbar, or every t >= i in full
// mode) is formed as a running product over t (the zeta products of Alg. 2) and
// its vector-Jacobian products are accumulated into step i.  No reverse
// recurrence and no tail identity are used, so the work is
// O(b * (tbar T - tbar (tbar - 1) / 2) * D * N) -- the paper's count of
// independent VJPs -- against O(b T D N) for the adjoint scan of the fused
// gradient kernel.  The results equal those of ssm_adjoint_grad up to rounding.
//
// Kernels:
//   k_pairs_pre : Delta (softplus of Delta_pre when asked) and g (the upstream
//                 gradient through the SiLU gate) per (step, channel), fp32;
//   k_chunk_aggr, k_carry (scan_kernels.h): the state carried into every chunk;
//   k_pairs     : one lane per (8 steps i, channel, 8 states), all pairs (t, i) of the window:
//                 the sum over t of lambda^{t,i} for the channel's states, into
//                 a [b][T][D][16] buffer (pairs of different i are independent);
//   k_pairs_epi : one lane per channel with its states in registers, the steps
//                 of one chunk in order: the forward state from the chunk's
//                 carry, the vjp epilogue with the summed lambda, per-block
//                 channel sums of dB, dC, and dL/dh0 from the pairs (t, -1);
//   k_reduce_bc, k_reduce_da1, k_reduce_da2 (scan_kernels.h): fixed-order sums.
#include "scan_kernels.h"

namespace ssmk {
namespace {

constexpr int kPairLanes = 64;  // channels per block (one wave)

// Delta and g per (step, channel) into dl / g ([b][T][D] fp32).
template <typename TI, bool SP, bool GATE>
__global__ __launch_bounds__(256) void k_pairs_pre(const ScanProblem p, float* dl, float* g) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= p.nb * p.T * p.D) return;
    const float pr = ldf(static_cast<const TI*>(p.delta), i);
    dl[i] = SP ? softplus_f(pr) : pr;
    const float dy = ldf(static_cast<const TI*>(p.dy), i);
    if constexpr (GATE) {
        const float zv = ldf(static_cast<const TI*>(p.z), i);
        g[i] = dy * zv * sigmoid_f(zv);
    } else {
        g[i] = dy;
    }
}

// grid (2 ceil(T/8), ceil(D/64), b), 64 threads: lane = channel, the wave one half of
// the states (8 of 16) for the steps i0 .. i0+7.
// mu[((b T + i) D + d) 16 + n] = sum_{t=i}^{min(T, i+W)-1} g_t C_t[n] P(i, t) with
// P(i, i) = 1 and P(i, t) = P(i, t-1) a_t, built as the running product of every i.
// The steps i share what depends on t alone: the loads of g_t, Delta_t and C_t, the
// exponential of a_t and the product g_t C_t are made once for eight pairs, which
// leaves one multiply and one FMA per pair and state (one step per wave: also an
// exponential, 8 cycles, and two more multiplies; 8.9 -> 3.1 ms at T = 4,096, b = 2,
// D = 1,536, W = 256).  Eight steps of eight states hold 128 registers of P and m (two
// waves per SIMD); four steps of 16 states would share each exponential by four only.
// The order of every sum and product is that of one step per lane.
constexpr int kPairSteps = 8;   // steps i per wave
constexpr int kPairStates = 8;  // states per lane

template <typename TI, bool N16>
__global__ __launch_bounds__(kPairLanes) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_pairs(
    const ScanProblem p, const float* dlv, const float* gv, float* mu, int64_t W) {
    constexpr int IB = kPairSteps, NS = kPairStates;
    // steps t loaded ahead of their use: four where a step's C is four registers (bf16, 16
    // states), two where it is eight (four there spilled 13 registers)
    constexpr int PB = N16 && sizeof(TI) == 2 ? 4 : 2;
    using Bits = typename RawIn<TI, 1>::Bits;
    const int lane = threadIdx.x;
    const int64_t d = static_cast<int64_t>(blockIdx.y) * kPairLanes + lane;
    const int half = blockIdx.x & 1, n0 = half * NS;
    const int64_t i0 = static_cast<int64_t>(blockIdx.x >> 1) * IB, bb = blockIdx.z;
    if (d >= p.D) return;
    if constexpr (!N16) {
        // at most 8 states: the other half's sums are zero (wave-uniform; with its pairs run
        // over zeros 4.24 -> 4.04 ms at b = 2, T = 4,096, D = 1,536, N = 8, W = 256, bf16; fp32 at
        // b = 2, T = 2,048, D = 768 1.28 -> 1.16).  The half that remains waits for its loads
        // of C, one per state and step.
        if (n0 >= p.N) {
            for (int u = 0; u < IB && i0 + u < p.T; ++u) {
                float4* o = reinterpret_cast<float4*>(mu + ((bb * p.T + i0 + u) * p.D + d) * 16 + n0);
                o[0] = o[1] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
            return;
        }
    }
    float cn[NS], P[IB][NS], m[IB][NS];
#pragma unroll
    for (int n = 0; n < NS; ++n) {
        const bool nv = n0 + n < p.N;
        const float al = nv ? p.A_log[p.ascalar ? d : d * p.N + n0 + n] : 0.f;
        cn[n] = nv ? -__expf(al) * kLog2e : 0.f;
#pragma unroll
        for (int u = 0; u < IB; ++u) {
            P[u][n] = 1.f;
            m[u][n] = 0.f;
        }
    }
    const int64_t rowb = bb * p.T;
    const TI* Cp = static_cast<const TI*>(p.C);
    const int64_t te = min(p.T, i0 + IB - 1 + W);  // past the last window's end
    // steps before `lo` or from `hi` on belong to the windows of some of the i only
    const int64_t lo = i0 + IB, hi = min(p.T, i0 + W);
    // the next PB steps' g, Delta and raw C (past the end: the last step again, not used)
    struct Batch {
        float g[PB], dl[PB];
        Bits c[N16 ? 1 : PB][NS];
        uint32_t cw[N16 ? PB : 1][sizeof(TI) * NS / 4];
    };
    auto load = [&](int64_t tb, Batch& o) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            const int64_t row = rowb + min(tb + u, te - 1);
            o.g[u] = gv[row * p.D + d];
            o.dl[u] = dlv[row * p.D + d];
            if constexpr (N16) {
                const uint4* src = reinterpret_cast<const uint4*>(Cp + row * 16 + n0);
#pragma unroll
                for (int q = 0; q < static_cast<int>(sizeof(TI)) / 2; ++q) {  // 16-byte pieces
                    const uint4 w = src[q];
                    o.cw[u][4 * q] = w.x;
                    o.cw[u][4 * q + 1] = w.y;
                    o.cw[u][4 * q + 2] = w.z;
                    o.cw[u][4 * q + 3] = w.w;
                }
            } else {
#pragma unroll
                for (int n = 0; n < NS; ++n) o.c[u][n] = n0 + n < p.N ? ldbits(Cp, row * p.N + n0 + n) : Bits(0);
            }
        }
    };
    auto cval = [&](const Batch& o, int u, int n) __attribute__((always_inline)) {
        uint32_t b;
        if constexpr (!N16) b = sizeof(TI) == 2 ? static_cast<uint32_t>(o.c[u][n]) << 16 : static_cast<uint32_t>(o.c[u][n]);
        else if constexpr (sizeof(TI) == 2) b = (n & 1) ? (o.cw[u][n >> 1] & 0xffff0000u) : (o.cw[u][n >> 1] << 16);
        else b = o.cw[u][n];
        return __uint_as_float(b);
    };
    // what step t gives every pair: a_t and g_t C_t
    float a[NS], gc[NS];
    auto shared = [&](const Batch& o, int s) __attribute__((always_inline)) {
        decays(cn, o.dl[s], a);
#pragma unroll
        for (int n = 0; n < NS; ++n) gc[n] = o.g[s] * cval(o, s, n);
    };
    Batch nx;
    load(i0, nx);
    int64_t tb = i0;
    // batches with a step that is not in every window, up to `end`
    auto edges = [&](int64_t end) __attribute__((always_inline)) {
#pragma unroll 1
        for (; tb < end; tb += PB) {
            const Batch cu = nx;
            load(tb + PB, nx);
#pragma unroll
            for (int s = 0; s < PB; ++s) {
                shared(cu, s);
#pragma unroll
                for (int u = 0; u < IB; ++u) {
                    // steps past the end and pairs outside the window change nothing, and the
                    // product starts at distance 1
                    const int64_t k = tb + s - (i0 + u);
                    const bool in = k >= 0 && k < W && tb + s < te, dec = in && k > 0;  // wave-uniform
#pragma unroll
                    for (int n = 0; n < NS; ++n) {
                        P[u][n] = dec ? P[u][n] * a[n] : P[u][n];
                        m[u][n] = in ? fmaf(gc[n], P[u][n], m[u][n]) : m[u][n];
                    }
                }
            }
        }
    };
    edges(min(lo, te));
#pragma unroll 1
    for (; tb + PB <= hi; tb += PB) {
        const Batch cu = nx;
        load(tb + PB, nx);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < PB; ++s) {
            shared(cu, s);
#pragma unroll
            for (int u = 0; u < IB; ++u)
#pragma unroll
                for (int n = 0; n < NS; ++n) {
                    P[u][n] *= a[n];
                    m[u][n] = fmaf(gc[n], P[u][n], m[u][n]);
                }
        }
    }
    edges(te);
#pragma unroll
    for (int u = 0; u < IB; ++u) {
        if (i0 + u >= p.T) break;
        float4* o = reinterpret_cast<float4*>(mu + ((rowb + i0 + u) * p.D + d) * 16 + n0);
        o[0] = make_float4(m[u][0], m[u][1], m[u][2], m[u][3]);
        o[1] = make_float4(m[u][4], m[u][5], m[u][6], m[u][7]);
    }
}

// grid (ceil(D/64), nc, b), 64 threads.  hbuf holds the state carried into each
// chunk on entry and receives the chunk's dA_log partial (dA * wn) on exit, at
// the same index.  The walk is serial, so a step's inputs are loaded a step ahead and
// the 32 channel sums are 16-byte LDS reads over all lanes (64 reads by half the lanes,
// next to the loads: 417 -> 258 us at T = 4,096, b = 2, D = 1,536).
template <typename TI, bool SP, bool GATE, bool N16>
__global__ __launch_bounds__(kPairLanes) void k_pairs_epi(const ScanProblem p, const float* dlv,
                                                           const float* gv, const float* mu) {
    __shared__ __attribute__((aligned(16))) float red[32][kPairLanes + 4];  // [dB, dC state][channel]
    const int lane = threadIdx.x;
    const int64_t d = static_cast<int64_t>(blockIdx.x) * kPairLanes + lane;
    const int64_t c = blockIdx.y, bb = blockIdx.z;
    const bool dv = d < p.D;
    const int64_t dd = dv ? d : 0;  // padding lanes read channel 0 and write nothing
    const TI* X = static_cast<const TI*>(p.x);
    const TI* DY = static_cast<const TI*>(p.dy);
    const TI* Z = static_cast<const TI*>(p.z);
    const TI* Bp = static_cast<const TI*>(p.B);
    const TI* Cp = static_cast<const TI*>(p.C);
    float cn[16], wn[16], h[16], dA[16];
    const int64_t cb = ((bb * p.nc + c) * p.N) * p.D + dd;
#pragma unroll
    for (int n = 0; n < 16; ++n) {
        const bool nv = n < p.N;
        const float al = nv ? p.A_log[p.ascalar ? dd : dd * p.N + n] : 0.f;
        const float e = nv ? __expf(al) : 0.f;
        wn[n] = -e;
        cn[n] = -e * kLog2e;
        h[n] = nv ? p.hbuf[cb + n * p.D] : 0.f;
        dA[n] = 0.f;
    }
    const int64_t rowb = bb * p.T;  // first row of this batch entry
    // dL/dh0 (full gradient): the pairs (t, -1), P(-1, t) = prod_{j=0}^{t} a_j
    if (p.dh0 && c == 0) {
        float P[16], m[16];
#pragma unroll
        for (int n = 0; n < 16; ++n) {
            P[n] = 1.f;
            m[n] = 0.f;
        }
        for (int64_t t = 0; t < p.T; ++t) {
            const int64_t td = (rowb + t) * p.D + dd;
            const float gt = gv[td], dlt = dlv[td];
            float Ct[16];
            ld_row16(Cp, rowb + t, p.N, Ct);
#pragma unroll
            for (int n = 0; n < 16; ++n) {
                P[n] *= fexp2(cn[n] * dlt);
                m[n] = fmaf(gt * Ct[n], P[n], m[n]);
            }
        }
        if (dv)
            for (int n = 0; n < p.N; ++n) p.dh0[(bb * p.D + d) * p.N + n] = m[n];
    }
    const int64_t t0 = c * p.L, t1 = min(t0 + p.L, p.T);
    const int64_t bsz = p.nb * p.T * p.N;
    float* pB = p.pB + static_cast<int64_t>(blockIdx.x) * bsz;
    float* pC = p.pC + static_cast<int64_t>(blockIdx.x) * bsz;
    // step i's inputs, loaded one step ahead (the last step reloads its own)
    struct In {
        float dl, g, dy, z, x;
        float4 lam[4];
        SRow<TI, N16> B, C;
    };
    auto load = [&](int64_t i, In& o) __attribute__((always_inline)) {
        const int64_t td = (rowb + i) * p.D + dd;
        o.dl = dlv[td];
        o.g = gv[td];
        o.x = ldf(X, td);
        o.dy = GATE ? ldf(DY, td) : 0.f;
        o.z = GATE ? ldf(Z, td) : 0.f;
        const float4* mi = reinterpret_cast<const float4*>(mu + td * 16);
#pragma unroll
        for (int q = 0; q < 4; ++q) o.lam[q] = mi[q];
        o.B.load(Bp, rowb + i, p.N);
        o.C.load(Cp, rowb + i, p.N);
    };
    // lane l adds 32 channels of sum l / 2, lane l ^ 1 the others
    const int ro = lane >> 1, rh = (lane & 1) * 32;
    In nx;
    load(t0, nx);
    for (int64_t i = t0; i < t1; ++i) {
        const In cu = nx;
        load(min(i + 1, t1 - 1), nx);
        __builtin_amdgcn_sched_barrier(0);
        const int64_t td = (rowb + i) * p.D + dd;
        const float dl = cu.dl, g = cu.g, xr = cu.x;
        const float xs = p.bdelta ? xr * dl : xr;  // the input term is (Delta) B x
        const float lam[16] = {cu.lam[0].x, cu.lam[0].y, cu.lam[0].z, cu.lam[0].w, cu.lam[1].x, cu.lam[1].y,
                               cu.lam[1].z, cu.lam[1].w, cu.lam[2].x, cu.lam[2].y, cu.lam[2].z, cu.lam[2].w,
                               cu.lam[3].x, cu.lam[3].y, cu.lam[3].z, cu.lam[3].w};
        float ah[16], y = 0.f;
        decays(cn, dl, ah);
#pragma unroll
        for (int n = 0; n < 16; ++n) {
            ah[n] *= h[n];  // a_i h_{i-1}
            h[n] = fmaf(cu.B.at(n), xs, ah[n]);
            y = fmaf(cu.C.at(n), h[n], y);
        }
        float dxp = 0.f, ddp = 0.f;
        wave_lds_sync();
#pragma unroll
        for (int n = 0; n < 16; ++n) {
            dxp = fmaf(lam[n], cu.B.at(n), dxp);
            const float s = lam[n] * ah[n];
            ddp = fmaf(s, wn[n], ddp);
            dA[n] = fmaf(s, dl, dA[n]);
            red[n][lane] = dv ? lam[n] * xs : 0.f;      // dB_i[n] over channels
            red[16 + n][lane] = dv ? g * h[n] : 0.f;    // dC_i[n] over channels
        }
        // with the Delta-scaled input, dx' = sum_n lambda B gives dx = dx' Delta and
        // adds dx' x to dDelta
        const float dd0 = p.bdelta ? fmaf(dxp, xr, ddp) : ddp;
        if (dv) {
            p.dx[td] = p.bdelta ? dxp * dl : dxp;
            p.ddelta[td] = SP ? dd0 * (1.f - fexp(-dl)) : dd0;  // d softplus / d Delta_pre
            if constexpr (GATE) {
                const float sg = sigmoid_f(cu.z);
                p.dz[td] = cu.dy * sg * (1.f + cu.z * (1.f - sg)) * y;
            }
        }
        wave_lds_sync();
        float4 s4 = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float4 v = *reinterpret_cast<const float4*>(&red[ro][rh + 4 * q]);
            s4.x += v.x;
            s4.y += v.y;
            s4.z += v.z;
            s4.w += v.w;
        }
        float sum = (s4.x + s4.y) + (s4.z + s4.w);
        sum += dpp_swap1(sum);
        if ((lane & 1) == 0 && (ro & 15) < p.N) (ro < 16 ? pB : pC)[(rowb + i) * p.N + (ro & 15)] = sum;
    }
    if (dv)
        for (int n = 0; n < p.N; ++n) p.hbuf[cb + n * p.D] = dA[n] * wn[n];
}

template <typename TI, bool SP, bool GATE>
hipError_t pairs_impl(const ScanProblem& p, float* dl, float* g, float* mu, int64_t W, hipStream_t s) {
    const int64_t MD = p.nb * p.T * p.D;
    {
        SSMK_TIMED("pairs_pre", s);
        hipLaunchKernelGGL((k_pairs_pre<TI, SP, GATE>), dim3(cdiv(MD, 256)), dim3(256), 0, s, p, dl, g);
    }
    {
        SSMK_TIMED("chunk_aggr", s);
        if (aggr_quad(p))
            hipLaunchKernelGGL((k_chunk_aggr_quad<TI, SP, GATE, false, 8>), aggr_grid(p), dim3(256), 0, s, p);
        else if (p.N == 16)
            hipLaunchKernelGGL((k_chunk_aggr<TI, SP, GATE, false, true, 8>), aggr_grid(p), dim3(64), 0, s, p);
        else
            hipLaunchKernelGGL((k_chunk_aggr<TI, SP, GATE, false, false, 8>), aggr_grid(p), dim3(64), 0, s, p);
    }
    {
        SSMK_TIMED("carry", s);
        hipLaunchKernelGGL(k_carry, carry_grid(p), dim3(256), 0, s, p);
    }
    {
        SSMK_TIMED("pairs", s);
        dim3 gp(2 * cdiv(p.T, kPairSteps), cdiv(p.D, kPairLanes), static_cast<unsigned>(p.nb));
        if (p.N == 16) hipLaunchKernelGGL((k_pairs<TI, true>), gp, dim3(kPairLanes), 0, s, p, dl, g, mu, W);
        else hipLaunchKernelGGL((k_pairs<TI, false>), gp, dim3(kPairLanes), 0, s, p, dl, g, mu, W);
    }
    {
        SSMK_TIMED("pairs_epilogue", s);
        dim3 ge(cdiv(p.D, kPairLanes), static_cast<unsigned>(p.nc), static_cast<unsigned>(p.nb));
        if (p.N == 16) hipLaunchKernelGGL((k_pairs_epi<TI, SP, GATE, true>), ge, dim3(kPairLanes), 0, s, p, dl, g, mu);
        else hipLaunchKernelGGL((k_pairs_epi<TI, SP, GATE, false>), ge, dim3(kPairLanes), 0, s, p, dl, g, mu);
    }
    SSMK_TIMED("reduce", s);
    hipLaunchKernelGGL(k_reduce_bc, dim3(cdiv(p.nb * p.T * p.N, 256)), dim3(256), 0, s, p);
    hipLaunchKernelGGL(k_reduce_da1, dim3(cdiv(p.D, 256), static_cast<unsigned>(p.N), static_cast<unsigned>(p.nslice)),
                       dim3(256), 0, s, p);
    hipLaunchKernelGGL(k_reduce_da2, dim3(cdiv(p.D * p.N, 256)), dim3(256), 0, s, p);
    return hipGetLastError();
}

template <typename TI>
hipError_t pairs_sel(const ScanProblem& p, float* dl, float* g, float* mu, int64_t W, hipStream_t s) {
    if (p.softplus) {
        if (p.gate) return pairs_impl<TI, true, true>(p, dl, g, mu, W, s);
        return pairs_impl<TI, true, false>(p, dl, g, mu, W, s);
    }
    if (p.gate) return pairs_impl<TI, false, true>(p, dl, g, mu, W, s);
    return pairs_impl<TI, false, false>(p, dl, g, mu, W, s);
}

size_t up256(size_t v) { return (v + 255) & ~static_cast<size_t>(255); }

}  // namespace

PairsWorkspace pairs_workspace(int64_t nb, int64_t T, int64_t D, int64_t N, int64_t L) {
    PairsWorkspace w{};
    const int64_t nc = (T + L - 1) / L;
    const int64_t nblk = (D + kPairLanes - 1) / kPairLanes;
    size_t off = 0;
    w.off_hbuf = off;
    off = up256(off + static_cast<size_t>(nb * nc * N * D) * sizeof(float));
    w.off_sdel = off;
    off = up256(off + static_cast<size_t>(nb * nc * D) * sizeof(double));
    w.off_dl = off;
    off = up256(off + static_cast<size_t>(nb * T * D) * sizeof(float));
    w.off_g = off;
    off = up256(off + static_cast<size_t>(nb * T * D) * sizeof(float));
    w.off_mu = off;
    off = up256(off + static_cast<size_t>(nb * T * D * 16) * sizeof(float));
    w.off_pB = off;
    off = up256(off + static_cast<size_t>(nblk * nb * T * N) * sizeof(float));
    w.off_pC = off;
    off = up256(off + static_cast<size_t>(nblk * nb * T * N) * sizeof(float));
    w.off_dAtmp = off;
    off = up256(off + static_cast<size_t>(choose_nslice(nb, nc)) * N * D * sizeof(float));
    w.total = off;
    return w;
}

hipError_t launch_grad_pairs(ScanProblem& p, void* ws, const PairsWorkspace& w, int64_t W, hipStream_t s) {
    char* b = static_cast<char*>(ws);
    p.hbuf = reinterpret_cast<float*>(b + w.off_hbuf);
    p.mbuf = nullptr;
    p.hseg = nullptr;
    p.cseg = nullptr;
    p.sdel = reinterpret_cast<double*>(b + w.off_sdel);
    p.psum = nullptr;
    p.pB = reinterpret_cast<float*>(b + w.off_pB);
    p.pC = reinterpret_cast<float*>(b + w.off_pC);
    p.dAtmp = reinterpret_cast<float*>(b + w.off_dAtmp);
    p.sink = nullptr;
    p.nsplit = static_cast<int>((p.D + kPairLanes - 1) / kPairLanes);
    p.nslice = choose_nslice(p.nb, p.nc);
    p.Dp = padded_channels(p.D);
    p.seg = grad_segment(p.L);
    p.dd16 = p.dz16 = p.bc16 = nullptr;
    float* dl = reinterpret_cast<float*>(b + w.off_dl);
    float* g = reinterpret_cast<float*>(b + w.off_g);
    float* mu = reinterpret_cast<float*>(b + w.off_mu);
    return p.bf16 ? pairs_sel<uint16_t>(p, dl, g, mu, W, s) : pairs_sel<float>(p, dl, g, mu, W, s);
}

}  // namespace ssmk
