// unstructured.hip -- the adjoint gradient of the unstructured SSM of Table 1
// (gfx950): an N = 16 state shared by the P channels, with per-step matrices
//   h_t = A_t h_{t-1} + B_t x_t,   y_t = C_t h_t,
//   A_t [N][N], B_t [N][P], C_t [P][N] (fp32, row-major), L = sum <dy_t, y_t>.
// Outputs: dA_t = mu_t h_{t-1}^T, dB_t = mu_t x_t^T, dx_t = B_t^T mu_t,
// dC_t = dy_t h_t^T (never truncated), dh0 = A_0^T mu_0 (full mode), where mu is
// the state cotangent mu_t = C_t^T dy_t + A_{t+1}^T mu_{t+1} (Prop. 1, summed over
// the loss terms as in Prop. 2), or in truncated mode the windowed adjoint of
// Eq. "capped", mubar_i = sum_{t=i}^{i+tbar-1} (A_{i+1}^T ... A_t^T) C_t^T dy_t.
//
// The state is tiny (16 values per sequence), so the parallelism comes from
// time: the sequence is cut into chunks of L steps, one wave per chunk.
//   k_un_aggr  : per chunk, the transition product Phi_c = A_e ... A_s (16x16x16
//                products on fp32 MFMA), the local end state from zero, the
//                local adjoint aggregate sum_t (A_t ... A_s)^T v_t and the
//                readout cotangents v_t = C_t^T dy_t of every step;
//   k_un_carry : per sequence, the chunk carries H_{c+1} = Phi_c H_c + hloc_c
//                and M_{c-1} = Phi_c^T M_c + mloc_c, in order;
//   k_un_wpre, k_un_wsuf : truncated mode.  The windowed adjoint obeys
//                mubar_i = u_i + A_{i+1}^T mubar_{i+1} with u_i = v_i - w_i and
//                w_i = Phi(i, i+tbar)^T v_{i+tbar}, Phi(i, j) = A_j ... A_{i+1} (the
//                step that leaves the window is taken out as it leaves), so it is
//                the full gradient's recurrence with v replaced by u.  w_i splits
//                at the block boundary k (blocks of tbar steps, i < k <= i + tbar):
//                w_i = Phi(i, k)^T y_{i+tbar} with y_j = Phi(k, j)^T v_j; k_un_wpre
//                runs the prefix products Phi(k, j) of each block and writes y,
//                k_un_wsuf the suffix products Phi(i, k)^T and writes u = v - w
//                over v; both keep the 16 x 16 products in MFMA registers;
//   k_un_madj  : truncated mode, each chunk's adjoint aggregate of u (the full
//                mode forms it inside k_un_aggr from v);
//   k_un_grad  : per chunk, the states recomputed from the carry (kept in LDS),
//                then the reverse sweep (or the windowed adjoints) and the vjps.
//   k_un_proj  : per step, the two reductions over the P channels that the
//                sequential passes need: bx_t = B_t x_t and v_t = C_t^T dy_t
//                (fully parallel, ahead of the chunk passes, so that these walk
//                only A_t and two 16-vectors per step).
// Lane layout of a wave: lane l = 16 q + i; the 16 x 16 matrices are held in the
// MFMA output layout (component r of lane (q, i): row 4q + r, column i) and the
// state vectors as such matrices with equal columns (component r: element 4q + r),
// so that a step's product needs no data movement between lanes (mul_vals, mul_vec).
// The passes over the steps are chains of dependent products.  What bounded them was
// the latency of each step's loads, one step ahead, and of the lane exchanges of the
// vector products; the loads now run 8 to 16 steps ahead (walk) and the vectors go
// through MFMA.  At b = 8, T = 16,384, P = 64, tbar = 256: k_un_wsuf 187 -> 72 us,
// k_un_wpre 96 -> 50, k_un_carry 82 -> 56, k_un_aggr 46 -> 43, k_un_madj 42 -> 28; what
// is left there is the chain itself (a product is 64 cycles of MFMA latency and 128 of
// the matrix pipe, so passes sharing a launch, or a SIMD, only take turns: measured
// slower; the vector products' tree of sums, mul_vec, is 12 more instructions a step).
// k_un_proj (1.16 GB, 256 us) and k_un_grad (2.1 GB, 426 us) run at the rate of a plain
// copy, 4.5 and 4.9 TB/s.
#include "internal.h"

namespace ssmk {
namespace {

constexpr int UN = 16;  // state size

// Sum over the four quarters of the wave (lanes i, i+16, i+32, i+48), by row swaps: no
// LDS latency in the passes' chains.
__device__ __forceinline__ float qsum(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const uint32_t s = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(s, s, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

struct UnArgs {
    int64_t nb, T, P, L, nc, tbar;
    int trunc;
    const float* A;   // [b][T][16][16]
    const float* B;   // [b][T][16][P]
    const float* C;   // [b][T][P][16]
    const float* x;   // [b][T][P]
    const float* h0;  // [b][16] or null
    const float* dy;  // [b][T][P]
    float* dA;
    float* dB;
    float* dC;
    float* dx;
    float* dh0;       // [b][16] or null (full mode)
    // workspace
    float* phi;       // [b][nc][16][16]
    float* hc;        // [b][nc][16]: local end state, then the carry into the chunk
    float* mc;        // [b][nc][16]: local adjoint aggregate, then the carry from the right
    float* v;         // [b][T][16]: C_t^T dy_t
    float* y;         // [b][T][16]: y_j = Phi(k, j)^T v_j (truncated mode)
    float* bx;        // [b][T][16]: B_t x_t
};

// grid (ceil(T / 4), b), 64 threads: four steps per wave, one at a time.
// bx_t = B_t x_t: instruction j reads rows 4j..4j+3 of B_t (row 4j + g in lanes
// 16 g .. 16 g + 15, four channels per lane, 64 channels per pass), and each
// row's partial sums are added over its 16 lanes.  v_t = C_t^T dy_t: lane l reads
// C_t[p][4(l%4) .. +3] for p = l/4 + 16 k (64 lanes cover 16 rows of C_t per
// pass), weighted by dy_t[p], and the 16 lanes with the same l%4 are added.
// Reads of B_t and C_t are contiguous across the wave.
__global__ __launch_bounds__(64) void k_un_proj(const UnArgs a) {
    const int lane = threadIdx.x, g = lane >> 4, sub = lane & 15, cq = lane & 3;
    const int64_t bb = blockIdx.y, P = a.P;
    for (int w = 0; w < 4; ++w) {
        const int64_t t = static_cast<int64_t>(blockIdx.x) * 4 + w;
        if (t >= a.T) return;  // wave-uniform
        const int64_t row = bb * a.T + t;
        const float* Bt = a.B + row * UN * P;
        const float* xt = a.x + row * P;
        const float* Ct = a.C + row * P * UN;
        const float* dyt = a.dy + row * P;
        float sb[4] = {0.f, 0.f, 0.f, 0.f};
        for (int64_t p = 4 * sub; p < P; p += 64) {
            const float4 x4 = *reinterpret_cast<const float4*>(xt + p);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 b4 = *reinterpret_cast<const float4*>(Bt + (4 * j + g) * P + p);
                sb[j] = fmaf(b4.x, x4.x, fmaf(b4.y, x4.y, fmaf(b4.z, x4.z, fmaf(b4.w, x4.w, sb[j]))));
            }
        }
        float sc[4] = {0.f, 0.f, 0.f, 0.f};
        for (int64_t pr = lane >> 2; pr < P; pr += 16) {
            const float4 c4 = *reinterpret_cast<const float4*>(Ct + pr * UN + 4 * cq);
            const float d = dyt[pr];
            sc[0] = fmaf(c4.x, d, sc[0]);
            sc[1] = fmaf(c4.y, d, sc[1]);
            sc[2] = fmaf(c4.z, d, sc[2]);
            sc[3] = fmaf(c4.w, d, sc[3]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            for (int m = 1; m < 16; m <<= 1) sb[j] += __shfl_xor(sb[j], m);
            for (int m = 4; m < 64; m <<= 1) sc[j] += __shfl_xor(sc[j], m);
        }
        // lane 16 g + 0 holds bx rows 4j + g; lanes 0..3 hold v[4 cq + j]
        if (sub == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) a.bx[row * UN + 4 * j + g] = sb[j];
        }
        if (lane < 4) {
#pragma unroll
            for (int j = 0; j < 4; ++j) a.v[row * UN + 4 * cq + j] = sc[j];
        }
    }
}

typedef float f4 __attribute__((ext_vector_type(4)));

// M X for a 16 x 16 matrix M and X in the MFMA output layout (lane 16 g + j holds
// X[4g + r][j] in component r): the four v_mfma_f32_16x16x4_f32 of the product
// each take, in lane 16 q + i, M[i][4q + kb] and X[4q + kb][i] (so instruction kb
// sums over the columns 4q + kb of M), and the latter is component kb of the
// lane's own X: the product needs no data movement and its result is again in
// the output layout.  m4 holds the lane's operand values of M (M[i][4q + kb], a
// float4 of row i; M[4q + kb][i] for M^T X, see vals_t), loaded ahead by the
// caller.  Two chains of two instructions (each waits for the one before it).
__device__ __forceinline__ f4 mul_vals(const float4 m4, f4 X) {
    f4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
    a = __builtin_amdgcn_mfma_f32_16x16x4f32(m4.x, X[0], a, 0, 0, 0);
    b = __builtin_amdgcn_mfma_f32_16x16x4f32(m4.z, X[2], b, 0, 0, 0);
    a = __builtin_amdgcn_mfma_f32_16x16x4f32(m4.y, X[1], a, 0, 0, 0);
    b = __builtin_amdgcn_mfma_f32_16x16x4f32(m4.w, X[3], b, 0, 0, 0);
    return a + b;
}
// M x + add for a state or adjoint vector (all columns of X alike): the four sums of four
// products are added as a tree and `add` last.  The chains of mul_vals started from `add`
// are 12 adds a step fewer and round every partial sum at add's magnitude (states
// and adjoints against 64 bits: 12 and 8 % more error).
__device__ __forceinline__ f4 mul_vec(const float4 m4, f4 X, f4 add = f4{0.f, 0.f, 0.f, 0.f}) {
    const f4 z = {0.f, 0.f, 0.f, 0.f};
    const f4 p0 = __builtin_amdgcn_mfma_f32_16x16x4f32(m4.x, X[0], z, 0, 0, 0);
    const f4 p1 = __builtin_amdgcn_mfma_f32_16x16x4f32(m4.y, X[1], z, 0, 0, 0);
    const f4 p2 = __builtin_amdgcn_mfma_f32_16x16x4f32(m4.z, X[2], z, 0, 0, 0);
    const f4 p3 = __builtin_amdgcn_mfma_f32_16x16x4f32(m4.w, X[3], z, 0, 0, 0);
    return ((p0 + p1) + (p2 + p3)) + add;
}
// Lane 16 q + i's operand values of M^T X.
__device__ __forceinline__ float4 vals_t(const float* M, int i, int q) {
    return make_float4(M[(4 * q) * UN + i], M[(4 * q + 1) * UN + i], M[(4 * q + 2) * UN + i], M[(4 * q + 3) * UN + i]);
}
__device__ __forceinline__ f4 identity16(int i, int q) {
    f4 e;
    for (int r = 0; r < 4; ++r) e[r] = (4 * q + r == i) ? 1.f : 0.f;
    return e;
}

// Sum over the 16 lanes of each quarter of the wave (every lane gets it).
template <int ROR>
__device__ __forceinline__ float add_ror(float v) {
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x120 + ROR, 0xF, 0xF, true));
}
__device__ __forceinline__ float sum16(float v) { return add_ror<1>(add_ror<2>(add_ror<4>(add_ror<8>(v)))); }

__device__ __forceinline__ f4 vec4(const float4 v) { return f4{v.x, v.y, v.z, v.w}; }
__device__ __forceinline__ float dot4(f4 a, f4 b) { return a[0] * b[0] + a[1] * b[1] + a[2] * b[2] + a[3] * b[3]; }
__device__ __forceinline__ f4 ld4v(const float* p) { return vec4(*reinterpret_cast<const float4*>(p)); }
__device__ __forceinline__ void st4v(float* p, f4 v) { *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]); }

// step(k, load(k)) for k = 0 .. n-1 in order, the loads of 8 steps issued together
// while the 8 steps before them run (two register buffers used alternately; past the
// end step n-1 is loaded again and not used).
template <typename Rec, typename Load, typename Step>
__device__ __forceinline__ void walk(int64_t n, Load load, Step step) {
    constexpr int U = 8;
    Rec ra[U], rb[U];
    auto fill = [&](int64_t k, Rec (&r)[U]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = load(min(k + u, n - 1));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto run = [&](int64_t k, const Rec (&r)[U]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k + u < n) step(k + u, r[u]);
    };
    fill(0, ra);
    for (int64_t k = 0; k < n; k += 2 * U) {
        fill(k + U, rb);
        run(k, ra);
        if (k + U >= n) break;
        fill(k + 2 * U, ra);
        run(k + U, rb);
    }
}

// grid (nc, b), 64 threads
__global__ __launch_bounds__(64) void k_un_aggr(const UnArgs a) {
    const int lane = threadIdx.x, i = lane & 15, q = lane >> 4;
    const int64_t c = blockIdx.x, bb = blockIdx.y;
    const int64_t s0 = c * a.L, s1 = min(s0 + a.L, a.T);
    const int64_t r0 = bb * a.T + s0;
    f4 phi = identity16(i, q);
    f4 h = {0.f, 0.f, 0.f, 0.f};
    float m = 0.f;  // lane (q, j): the quarter's share of m[j]
    struct Rec {
        float4 A;
        f4 bx, v;
    };
    walk<Rec>(
        s1 - s0,
        [&](int64_t k) {
            const int64_t row = r0 + k;
            return Rec{*reinterpret_cast<const float4*>(a.A + row * UN * UN + i * UN + 4 * q), ld4v(a.bx + row * UN + 4 * q),
                       ld4v(a.v + row * UN + 4 * q)};
        },
        [&](int64_t, const Rec& r) {
            h = mul_vec(r.A, h, r.bx);  // h <- A_t h + B_t x_t
            phi = mul_vals(r.A, phi);    // Phi <- A_t Phi
            // the adjoint aggregate m += Phi_t^T v_t; lane (q, j): sum_r Phi[4q + r][j] v[4q + r]
            if (!a.trunc) m += dot4(phi, r.v);
        });
    const int64_t cb = bb * a.nc + c;
    for (int r = 0; r < 4; ++r) a.phi[cb * UN * UN + (4 * q + r) * UN + i] = phi[r];
    m = qsum(m);
    if (q == 0) a.mc[cb * UN + i] = m;
    if (i == 0) st4v(a.hc + cb * UN + 4 * q, h);
}

// grid (2 b), 64 threads: workgroup 2 bb + dir walks the chunks of sequence bb
// forwards (dir 0) or backwards (dir 1).  Each carry replaces the aggregate it has
// consumed (which was loaded before).
__global__ __launch_bounds__(64) void k_un_carry(const UnArgs a) {
    const int lane = threadIdx.x, i = lane & 15, q = lane >> 4;
    const int64_t bb = blockIdx.x >> 1;
    const int64_t nc = a.nc, c0 = bb * nc;
    struct Rec {
        float4 P;
        f4 loc;
    };
    f4 X = {0.f, 0.f, 0.f, 0.f};
    if (blockIdx.x & 1) {
        // M_{c-1} = Phi_c^T M_c + mloc_c
        walk<Rec>(
            nc,
            [&](int64_t k) {
                const int64_t cb = c0 + nc - 1 - k;
                return Rec{vals_t(a.phi + cb * UN * UN, i, q), ld4v(a.mc + cb * UN + 4 * q)};
            },
            [&](int64_t k, const Rec& r) {
                if (i == 0) st4v(a.mc + (c0 + nc - 1 - k) * UN + 4 * q, X);  // the carry from the right into the chunk
                X = mul_vec(r.P, X, r.loc);
            });
        if (a.dh0 && i == 0) st4v(a.dh0 + bb * UN + 4 * q, X);
        return;
    }
    // H_{c+1} = Phi_c H_c + hloc_c
    if (a.h0) X = ld4v(a.h0 + bb * UN + 4 * q);
    walk<Rec>(
        nc,
        [&](int64_t k) {
            const int64_t cb = c0 + k;
            return Rec{*reinterpret_cast<const float4*>(a.phi + cb * UN * UN + i * UN + 4 * q), ld4v(a.hc + cb * UN + 4 * q)};
        },
        [&](int64_t k, const Rec& r) {
            if (i == 0) st4v(a.hc + (c0 + k) * UN + 4 * q, X);  // the carry into the chunk
            X = mul_vec(r.P, X, r.loc);
        });
}

// grid (blocks - 1, b), 64 threads: block beta >= 1, steps [k, k + tbar) with
// k = beta tbar; Pre = Phi(k, j) = A_j ... A_{k+1} in registers (output layout),
// y_j = Pre^T v_j (lane (g, j'): sum_r Pre[4g + r][j'] v_j[4g + r], summed over g).
__global__ __launch_bounds__(64) void k_un_wpre(const UnArgs a) {
    const int lane = threadIdx.x, i = lane & 15, q = lane >> 4;
    const int64_t bb = blockIdx.y;
    const int64_t k = (static_cast<int64_t>(blockIdx.x) + 1) * a.tbar;
    if (k >= a.T) return;
    const int64_t r0 = bb * a.T + k;
    f4 pre = identity16(i, q);
    struct Rec {
        float4 A;
        f4 v;
    };
    walk<Rec>(
        min(a.tbar, a.T - k),
        [&](int64_t j) {
            const int64_t row = r0 + j;  // (A_k is loaded and not used)
            return Rec{*reinterpret_cast<const float4*>(a.A + row * UN * UN + i * UN + 4 * q), ld4v(a.v + row * UN + 4 * q)};
        },
        [&](int64_t j, const Rec& r) {
            if (j > 0) pre = mul_vals(r.A, pre);
            const float y = qsum(dot4(pre, r.v));
            if (q == 0) a.y[(r0 + j) * UN + i] = y;
        });
}

// grid (blocks, b), 64 threads: block beta, steps [beta tbar, k) with k =
// (beta + 1) tbar < T; S = Phi(i, k)^T = A_{i+1}^T S(i + 1), S(k) = I, in registers
// (output layout: lane (g, n) holds S[4g + r][n]); w_i = S y_{i+tbar} (lane (g, n):
// S[4g + r][n] y[n], summed over n), and v_i -= w_i while i + tbar < T.
__global__ __launch_bounds__(64) void k_un_wsuf(const UnArgs a) {
    const int lane = threadIdx.x, i = lane & 15, q = lane >> 4;
    const int64_t bb = blockIdx.y;
    const int64_t k = (static_cast<int64_t>(blockIdx.x) + 1) * a.tbar;
    if (k >= a.T) return;
    const int64_t base = bb * a.T;
    f4 sm = identity16(i, q);
    struct Rec {
        float4 A;
        f4 v;
        float y;
    };
    walk<Rec>(
        a.tbar,
        [&](int64_t j) {
            const int64_t t = k - 1 - j;  // a y past the end is not used
            return Rec{vals_t(a.A + (base + t + 1) * UN * UN, i, q), ld4v(a.v + (base + t) * UN + 4 * q),
                       a.y[(base + min(t + a.tbar, a.T - 1)) * UN + i]};
        },
        [&](int64_t j, const Rec& r) {
            const int64_t t = k - 1 - j;
            sm = mul_vals(r.A, sm);
            if (t + a.tbar >= a.T) return;  // wave-uniform
            f4 w;
#pragma unroll
            for (int c = 0; c < 4; ++c) w[c] = sum16(sm[c] * r.y);
            if (i == 0) st4v(a.v + (base + t) * UN + 4 * q, r.v - w);
        });
}

// grid (nc, b), 64 threads: the chunk's adjoint aggregate of u (v after
// k_un_wsuf), as k_un_aggr forms it from v in full mode: rho_e = u_e,
// rho_t = u_t + A_{t+1}^T rho_{t+1}, mloc = A_s^T rho_s.
__global__ __launch_bounds__(64) void k_un_madj(const UnArgs a) {
    const int lane = threadIdx.x, i = lane & 15, q = lane >> 4;
    const int64_t c = blockIdx.x, bb = blockIdx.y;
    const int64_t s0 = c * a.L, s1 = min(s0 + a.L, a.T);
    const int64_t re = bb * a.T + s1 - 1;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 carry = zero;  // A_{t+1}^T rho_{t+1}
    struct Rec {
        float4 A;
        f4 v;
    };
    walk<Rec>(
        s1 - s0, [&](int64_t j) { return Rec{vals_t(a.A + (re - j) * UN * UN, i, q), ld4v(a.v + (re - j) * UN + 4 * q)}; },
        [&](int64_t, const Rec& r) { carry = mul_vec(r.A, r.v + carry); });
    if (i == 0) st4v(a.mc + (bb * a.nc + c) * UN + 4 * q, carry);
}

// grid (nc, b), 256 threads: wave 0 walks the chunk's states h_{s-1} .. h_e into LDS,
// wave 1 its adjoints (each needs only its own carry); then the four waves write the
// vjps of the steps, independent of one another, four steps at a time.
constexpr int kUnGradWaves = 4;
template <int L>
__global__ __launch_bounds__(64 * kUnGradWaves) void k_un_grad(const UnArgs a) {
    __shared__ __attribute__((aligned(16))) float shs[L + 1][UN];
    __shared__ __attribute__((aligned(16))) float smu[L][UN];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, i = lane & 15, q = lane >> 4;
    const int64_t c = blockIdx.x, bb = blockIdx.y;
    const int64_t s0 = c * L, s1 = min(s0 + L, a.T);
    const int64_t cb = bb * a.nc + c;
    const int64_t r0 = bb * a.T + s0;
    const int n = static_cast<int>(s1 - s0);
    const int P = static_cast<int>(a.P);
    struct Rec {
        float4 A;
        f4 v;
    };
    if (wave == 0) {
        f4 h = ld4v(a.hc + cb * UN + 4 * q);
        if (i == 0) st4v(&shs[0][4 * q], h);
        walk<Rec>(
            n,
            [&](int64_t k) {
                const int64_t row = r0 + k;
                return Rec{*reinterpret_cast<const float4*>(a.A + row * UN * UN + i * UN + 4 * q), ld4v(a.bx + row * UN + 4 * q)};
            },
            [&](int64_t k, const Rec& r) {
                h = mul_vec(r.A, h, r.v);
                if (i == 0) st4v(&shs[k + 1][4 * q], h);
            });
    } else if (wave == 1) {
        // mu_t = v_t + A_{t+1}^T mu_{t+1}; in truncated mode v holds u and the recurrence
        // gives the windowed adjoint
        f4 mun = ld4v(a.mc + cb * UN + 4 * q);  // A_{t+1}^T mu_{t+1}
        walk<Rec>(
            n,
            [&](int64_t k) {
                const int64_t row = r0 + n - 1 - k;
                return Rec{vals_t(a.A + row * UN * UN, i, q), ld4v(a.v + row * UN + 4 * q)};
            },
            [&](int64_t k, const Rec& r) {
                const f4 mu = r.v + mun;
                if (i == 0) st4v(&smu[n - 1 - k][4 * q], mu);
                mun = mul_vec(r.A, mu);
            });
    }
    __syncthreads();
    // 256 consecutive values of dB_t and dC_t per pass: lane l's four start at row
    // r, column pb of dB_t (row pc, column rc of dC_t), moved on from pass to pass
    const int e0 = 4 * lane, er = e0 / P, ep = e0 - er * P, dr = 256 / P, dp = 256 - dr * P, rc = e0 % UN;
    for (int k = wave; k < n; k += kUnGradWaves) {
        const int64_t row = r0 + k;
        {
            // dA_t[r][4(l%4) .. +3] = mu[r] h_{t-1}[..], r = l / 4
            const int r = lane >> 2, c4 = (lane & 3) * 4;
            st4v(a.dA + row * UN * UN + e0, ld4v(&shs[k][c4]) * smu[k][r]);
        }
        // dB_t[r][p] = mu[r] x_t[p]; dC_t[p][r] = dy_t[p] h_t[r]
        const float* xt = a.x + row * P;
        const float* dyt = a.dy + row * P;
        float* dB = a.dB + row * UN * P;
        float* dC = a.dC + row * UN * P;
        const f4 hv = ld4v(&shs[k + 1][rc]);
        int r = er, pb = ep;
#pragma unroll 4
        for (int e = e0; e < UN * P; e += 256) {
            st4v(dB + e, ld4v(xt + pb) * smu[k][r]);
            st4v(dC + e, hv * dyt[e / UN]);
            r += dr;
            pb += dp;
            if (pb >= P) {
                pb -= P;
                ++r;
            }
        }
        // dx_t[p] = sum_r B_t[r][p] mu[r]
        const float* Bt = a.B + row * UN * P;
        for (int p = lane; p < P; p += 64) {
            float sx = 0.f;
#pragma unroll
            for (int rr = 0; rr < UN; ++rr) sx = fmaf(Bt[rr * P + p], smu[k][rr], sx);
            a.dx[row * P + p] = sx;
        }
    }
}

}  // namespace

size_t unstructured_workspace(int64_t nb, int64_t T, int64_t L, bool trunc) {
    const int64_t nc = (T + L - 1) / L;
    auto up = [](size_t v) { return (v + 255) & ~size_t(255); };
    size_t s = up(size_t(nb * nc) * UN * UN * 4) + 2 * up(size_t(nb * nc) * UN * 4) + 2 * up(size_t(nb * T) * UN * 4);
    if (trunc) s += up(size_t(nb * T) * UN * 4);
    return s;
}

hipError_t launch_unstructured_grad(const UnstructuredProblem& u, void* ws, hipStream_t s) {
    UnArgs a{};
    a.nb = u.nb;
    a.T = u.T;
    a.P = u.P;
    a.L = u.L;
    a.nc = (u.T + u.L - 1) / u.L;
    a.trunc = u.trunc ? 1 : 0;
    a.tbar = u.tbar;
    a.A = u.A;
    a.B = u.B;
    a.C = u.C;
    a.x = u.x;
    a.h0 = u.h0;
    a.dy = u.dy;
    a.dA = u.dA;
    a.dB = u.dB;
    a.dC = u.dC;
    a.dx = u.dx;
    a.dh0 = u.dh0;
    auto up = [](size_t v) { return (v + 255) & ~size_t(255); };
    char* w = static_cast<char*>(ws);
    a.phi = reinterpret_cast<float*>(w);
    w += up(size_t(a.nb * a.nc) * UN * UN * 4);
    a.hc = reinterpret_cast<float*>(w);
    w += up(size_t(a.nb * a.nc) * UN * 4);
    a.mc = reinterpret_cast<float*>(w);
    w += up(size_t(a.nb * a.nc) * UN * 4);
    a.v = reinterpret_cast<float*>(w);
    w += up(size_t(a.nb * a.T) * UN * 4);
    a.bx = reinterpret_cast<float*>(w);
    w += up(size_t(a.nb * a.T) * UN * 4);
    a.y = u.trunc ? reinterpret_cast<float*>(w) : nullptr;
    const dim3 gc(static_cast<unsigned>(a.nc), static_cast<unsigned>(a.nb));
    {
        SSMK_TIMED("un_proj", s);
        hipLaunchKernelGGL(k_un_proj, dim3(static_cast<unsigned>((a.T + 3) / 4), static_cast<unsigned>(a.nb)),
                           dim3(64), 0, s, a);
    }
    {
        SSMK_TIMED("un_aggr", s);
        hipLaunchKernelGGL(k_un_aggr, gc, dim3(64), 0, s, a);
    }
    if (a.trunc) {
        const int64_t nblk = (a.T + a.tbar - 1) / a.tbar;  // at least 2 (tbar < T)
        {
            SSMK_TIMED("un_wpre", s);
            hipLaunchKernelGGL(k_un_wpre, dim3(static_cast<unsigned>(nblk - 1), static_cast<unsigned>(a.nb)),
                               dim3(64), 0, s, a);
        }
        {
            SSMK_TIMED("un_wsuf", s);
            hipLaunchKernelGGL(k_un_wsuf, dim3(static_cast<unsigned>(nblk), static_cast<unsigned>(a.nb)), dim3(64),
                               0, s, a);
        }
        SSMK_TIMED("un_madj", s);
        hipLaunchKernelGGL(k_un_madj, gc, dim3(64), 0, s, a);
    }
    {
        SSMK_TIMED("un_carry", s);
        hipLaunchKernelGGL(k_un_carry, dim3(static_cast<unsigned>(2 * a.nb)), dim3(64), 0, s, a);
    }
    SSMK_TIMED("un_grad", s);
    switch (a.L) {
        case 16: hipLaunchKernelGGL(k_un_grad<16>, gc, dim3(64 * kUnGradWaves), 0, s, a); break;
        case 32: hipLaunchKernelGGL(k_un_grad<32>, gc, dim3(64 * kUnGradWaves), 0, s, a); break;
        case 64: hipLaunchKernelGGL(k_un_grad<64>, gc, dim3(64 * kUnGradWaves), 0, s, a); break;
        case 128: hipLaunchKernelGGL(k_un_grad<128>, gc, dim3(64 * kUnGradWaves), 0, s, a); break;
        default: hipLaunchKernelGGL(k_un_grad<256>, gc, dim3(64 * kUnGradWaves), 0, s, a); break;
    }
    return hipGetLastError();
}

}  // namespace ssmk
