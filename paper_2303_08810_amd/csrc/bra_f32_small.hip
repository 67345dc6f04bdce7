// float32 tensors, regions of 4 x 4 tokens, heads of 32 channels, at most 64 routed keys: the
// whole layer in two launches, all products on the float32 matrix-core instruction
// v_mfma_f32_16x16x4_f32 (lane 16 g + i holds A[row i][k g], B[k g][col i] and D[rows 4 g + j]
// [col i]; a lane that loads 4 consecutive floats of its row feeds 4 such products, the
// contraction index then runs over {16 s + 4 g' + e} in product e of step s: any order will do
// as long as both operands use the same one).
//
//   k_f32_qkv : workgroup = one region.  Q, K, V = X [Wq | Wk | Wv] (Eq. 3) of its 16 tokens, and
//               the sums of Q and K over them (Sec. 3.2: Q^r, K^r are the per-region means).
//   k_f32_attn: workgroup = one region.  Its row of A^r = Q^r (K^r)^T (Eq. 4) and the top-k of it
//               (Eq. 5), the gathered keys and values (Eq. 6), attention (Eq. 1), LCE (Eq. 7; 5 x 5
//               depth-wise correlation of V, zero padding) and W^o (Eq. 2).
//   k_f32_route: the same routing rows on their own, for routing-only calls.
#include "bra_mfma_dev.h"

namespace bra {

using namespace mfma;

namespace {

constexpr int kN = 16;       // tokens of a region
constexpr int kKeys = 64;    // keys of a region's attention at most

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// token (in the image) of slot q of region r
__device__ __forceinline__ int region_token(const Dims &D, int r, int q)
{
    const int gy = r / D.S, gx = r - gy * D.S;
    return (gy * 4 + q / 4) * D.W + gx * 4 + q % 4;
}

// SUMS: the sums of Q and K alone.
template <int C, bool SUMS>
__global__ __launch_bounds__(256) void k_f32_qkv(const float *__restrict__ X, const float *__restrict__ Wqkv,
                                                 float *__restrict__ QKV, float *__restrict__ Pq,
                                                 float *__restrict__ Pk, Dims D)
{
    const int b = blockIdx.x / D.R, r = blockIdx.x % D.R;
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int g = lane / 16, i = lane % 16;
    const size_t img = (size_t)b * D.N;
    const float *xrow = X + (img + region_token(D, r, i)) * C + 4 * g;
    f32x4 xa[C / 16];
#pragma unroll
    for (int s = 0; s < C / 16; ++s) xa[s] = *(const f32x4 *)(xrow + 16 * s);
    size_t orow[4];      // rows 4 g + j of the result
#pragma unroll
    for (int j = 0; j < 4; ++j) orow[j] = (img + region_token(D, r, 4 * g + j)) * 3 * C;
    // 16 output channels at a time: the weights of all a wavefront's tiles are requested before the first product
    constexpr int NT = (SUMS ? 2 : 3) * C / 64;
    float wb[NT][C / 16][4];
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int s = 0; s < C / 16; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) wb[u][s][e] = Wqkv[(size_t)(16 * s + 4 * g + e) * 3 * C + 16 * (wave + 4 * u) + i];
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        const int ct = wave + 4 * u;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < C / 16; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = mfma_f32(xa[s][e], wb[u][s][e], acc);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (!SUMS) QKV[orow[j] + 16 * ct + i] = acc[j];
        if (16 * ct < 2 * C) {      // Q and K: sums over the region's tokens, in a fixed order
            float v = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            if (g == 0) {
                float *dst = 16 * ct < C ? Pq : Pk;
                dst[((size_t)b * D.R + r) * C + (16 * ct) % C + i] = v;
            }
        }
    }
}

// Row r of A^r of image b from the region sums (entry j to aff[j], j < 64; entries past R are not
// meaningful), by 256 threads: 4 lanes per key region, a quarter of the channels each.  finish() ends with a
// barrier.
template <int C>
struct RouteRow {
    f32x4 q[C / 16], k[C / 16];
    __device__ __forceinline__ void request(const float *__restrict__ Pq_row, const float *__restrict__ Pk_img, int R)
    {
        const int jj = threadIdx.x / 4, cq = threadIdx.x % 4;
        const float *krow = Pk_img + (size_t)min(jj, R - 1) * C + cq * (C / 4);
        const float *qrow = Pq_row + cq * (C / 4);
#pragma unroll
        for (int c = 0; c < C / 16; ++c) {
            q[c] = *(const f32x4 *)(qrow + 4 * c);
            k[c] = *(const f32x4 *)(krow + 4 * c);
        }
    }
    __device__ __forceinline__ void finish(float sc, float *aff) const
    {
        float a = 0.f;
#pragma unroll
        for (int c = 0; c < C / 16; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) a = fmaf(q[c][e], k[c][e], a);
        a = dpp_fadd<0xB1>(a);
        a = dpp_fadd<0x4E>(a);
        if (threadIdx.x % 4 == 0) aff[threadIdx.x / 4] = a * sc;
        __syncthreads();
    }
};

template <int C>
__global__ __launch_bounds__(256) void k_f32_route(const float *__restrict__ Pq, const float *__restrict__ Pk,
                                                   int32_t *__restrict__ Ir, float *__restrict__ Ar, Dims D)
{
    __shared__ float aff[64];
    const int b = blockIdx.x / D.R, r = blockIdx.x % D.R;
    const size_t row = (size_t)b * D.R + r;
    const float inv_n = 1.0f / (float)kN;
    RouteRow<C> routing;
    routing.request(Pq + row * C, Pk + (size_t)b * D.R * C, D.R);
    routing.finish(inv_n * inv_n, aff);
    if (threadIdx.x < kWave) {
        const int lane = threadIdx.x;
        const float v = aff[lane];
        if (Ar && lane < D.R) Ar[row * D.R + lane] = v;
        wave_topk(v, lane, D.R, D.k, Ir + row * D.k);
    }
}

// Four wavefronts take a head each, with 64 channels half of its keys each: HALVES parts of every output.
template <int C>
struct F32Smem {
    static constexpr int P = C + 4;                       // floats per row of the tiles (4 x odd: conflict-free 16-byte reads of 16 rows)
    static constexpr int HEADS = C / 32, HALVES = 4 / HEADS;
    static constexpr size_t tile = (size_t)16 * P * 4;
    static constexpr size_t k_off = 0;
    static constexpr size_t v_off = k_off + 4 * tile;
    static constexpr size_t h_off = v_off + 4 * tile;                     // V over the region and a 2-token halo: 8 x 8 tokens
    static constexpr size_t q_off = h_off + 4 * tile;                     // Q, later the attention's parts
    static constexpr size_t l_off = q_off + HALVES * tile;                // LCE(V)
    static constexpr size_t t_off = l_off + tile;                         // LCE's taps [C][25]
    static constexpr size_t m_off = t_off + (size_t)C * 25 * 4;           // reference and denominator [HALVES][HEADS][16]
    static constexpr size_t a_off = m_off + (size_t)HALVES * HEADS * 16 * 8;      // affinities [64], routed regions [4]
    static constexpr size_t bytes = a_off + 64 * 4 + 16 * 4;
};

// The chain is routing row, top-k, gather, attention, W^o, with one workgroup per compute unit and nothing to hide it: what it waits
// for comes first in the order of requests (loads return in order), the convolution runs while the gather is on its way, and
// the softmax stays in registers (S^T = K Q^T: a lane has 16 or 8 keys of one query).  1 x 28 x 28 x 64: 10.6 -> 6.3
// us, 1 x 28 x 28 x 128 the layer 28.5 -> 17.9.
template <int C>
__global__ __launch_bounds__(256) void k_f32_attn(const float *__restrict__ QKV, const float *__restrict__ Pq,
                                                  const float *__restrict__ Pk, const int32_t *__restrict__ Ir_in,
                                                  int32_t *__restrict__ Ir_out, const float *__restrict__ Wlce,
                                                  const float *__restrict__ Wo, float *__restrict__ Y, Dims D)
{
    typedef F32Smem<C> SM;
    constexpr int P = SM::P, HEADS = SM::HEADS, HALVES = SM::HALVES, KT = kKeys / 16 / HALVES;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float *Ks = (float *)(smem + SM::k_off), *Vs = (float *)(smem + SM::v_off), *Hs = (float *)(smem + SM::h_off);
    float *Qs = (float *)(smem + SM::q_off), *Ls = (float *)(smem + SM::l_off), *Ts = (float *)(smem + SM::t_off);
    f32x2 *state = (f32x2 *)(smem + SM::m_off);
    float *aff = (float *)(smem + SM::a_off);
    int32_t *irs = (int32_t *)(aff + 64);

    const int b = blockIdx.x / D.R, r = blockIdx.x % D.R, tid = threadIdx.x;
    const int wave = tid / kWave, lane = tid % kWave;
    const int g = lane / 16, i = lane % 16;
    const size_t img = (size_t)b * D.N;
    const size_t row = (size_t)b * D.R + r;
    const int gy = r / D.S, gx = r - gy * D.S;
    const int y0 = 4 * gy, x0 = 4 * gx;
    const int kn = D.k * kN;

    // routing (Eq. 4, 5): given, or this region's row of A^r and its k largest entries
    RouteRow<C> routing;
    if (!Ir_in) routing.request(Pq + row * C, Pk + (size_t)b * D.R * C, D.R);
    // what does not depend on it: V over the halo and LCE's taps, Q, and the W^o operands of this wavefront's output tiles
    constexpr int C4 = C / 4;                              // 16-byte chunks of a row
    constexpr int NQ = 16 * C4 / 256, NH = 64 * C4 / 256, NW = (C * 25 / 4 + 255) / 256;
    f32x4 qreg[NQ], hreg[NH], treg[NW];
#pragma unroll
    for (int u = 0; u < NH; ++u) {
        const int idx = tid + 256 * u;
        const int t = idx / C4, y = y0 - 2 + t / 8, x = x0 - 2 + t % 8;
        const bool ok = (unsigned)y < (unsigned)D.H && (unsigned)x < (unsigned)D.W;
        hreg[u] = *(const f32x4 *)(QKV + (img + (ok ? y * D.W + x : 0)) * 3 * C + 2 * C + 4 * (idx % C4));
    }
#pragma unroll
    for (int u = 0; u < NW; ++u) treg[u] = *(const f32x4 *)(Wlce + 4 * min(tid + 256 * u, C * 25 / 4 - 1));
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int idx = tid + 256 * u;
        qreg[u] = *(const f32x4 *)(QKV + (img + region_token(D, r, idx / C4)) * 3 * C + 4 * (idx % C4));
    }
    constexpr int NOT = C / 64;                            // output-channel tiles of 16 per wavefront
    float wo[NOT][C / 16][4];
#pragma unroll
    for (int u = 0; u < NOT; ++u)
#pragma unroll
        for (int s = 0; s < C / 16; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) wo[u][s][e] = Wo[(size_t)(16 * s + 4 * g + e) * C + 16 * (wave + 4 * u) + i];
    __builtin_amdgcn_sched_barrier(0);

    if (Ir_in) {
        if (tid < D.k) irs[tid] = region_index(Ir_in[row * D.k + tid], D.R);
    } else {
        const float inv_n = 1.0f / (float)kN;
        routing.finish(inv_n * inv_n, aff);
        if (wave == 0) wave_topk(aff[lane], lane, D.R, D.k, irs);
    }
#pragma unroll
    for (int u = 0; u < NH; ++u) {
        const int idx = tid + 256 * u;
        const int t = idx / C4, y = y0 - 2 + t / 8, x = x0 - 2 + t % 8;
        const bool ok = (unsigned)y < (unsigned)D.H && (unsigned)x < (unsigned)D.W;
        *(f32x4 *)(Hs + t * P + 4 * (idx % C4)) = ok ? hreg[u] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int u = 0; u < NW; ++u)
        if (tid + 256 * u < C * 25 / 4) *(f32x4 *)(Ts + 4 * (tid + 256 * u)) = treg[u];
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int idx = tid + 256 * u;
        *(f32x4 *)(Qs + (idx / C4) * P + 4 * (idx % C4)) = qreg[u];
    }
    __syncthreads();
    if (Ir_out && tid < D.k) Ir_out[row * D.k + tid] = Ir_in ? Ir_in[row * D.k + tid] : irs[tid];

    // gathered keys and values (Eq. 6): key l is token l % 16 of routed region l / 16
    constexpr int NK = kKeys * C4 / 256;
    f32x4 kr[NK], vr[NK];
#pragma unroll
    for (int u = 0; u < NK; ++u) {
        const int idx = tid + 256 * u;
        const int key = min(idx / C4, kn - 1);      // rows past the end repeat the last key; masked below
        const float *src = QKV + (img + region_token(D, irs[key / kN], key % kN)) * 3 * C + 4 * (idx % C4);
        kr[u] = *(const f32x4 *)(src + C);
        vr[u] = *(const f32x4 *)(src + 2 * C);
    }
    __builtin_amdgcn_sched_barrier(0);
    // LCE (Eq. 7) meanwhile: thread = (channel, every (256 / C)-th column of the region)
    const int lc = tid % C;
    float tap[25];
#pragma unroll
    for (int t = 0; t < 25; ++t) tap[t] = Ts[lc * 25 + t];
#pragma unroll
    for (int v = 0; v < C / 64; ++v) {
        const int qx = tid / C + 256 / C * v;
        float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            float in[5];
#pragma unroll
            for (int kx = 0; kx < 5; ++kx) in[kx] = Hs[(y * 8 + qx + kx) * P + lc];
#pragma unroll
            for (int qy = 0; qy < 4; ++qy) {
                if (y < qy || y > qy + 4) continue;
#pragma unroll
                for (int kx = 0; kx < 5; ++kx) a[qy] = fmaf(tap[(y - qy) * 5 + kx], in[kx], a[qy]);
            }
        }
#pragma unroll
        for (int qy = 0; qy < 4; ++qy) Ls[(4 * qy + qx) * P + lc] = a[qy];
    }
    const int h = wave % HEADS, half = wave / HEADS;
    f32x4 qf[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) qf[s] = *(const f32x4 *)(Qs + i * P + 32 * h + 16 * s + 4 * g) * (D.scale * 1.4426950408889634f);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < NK; ++u) {
        const int idx = tid + 256 * u;
        *(f32x4 *)(Ks + (idx / C4) * P + 4 * (idx % C4)) = kr[u];
        *(f32x4 *)(Vs + (idx / C4) * P + 4 * (idx % C4)) = vr[u];
    }
    __syncthreads();

    // S^T[key 16 t + 4 g + j][query i] of this wavefront's keys, as exponents of 2
    const int key0 = kKeys / HALVES * half;
    f32x4 st[KT], kf[KT][2];
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int s = 0; s < 2; ++s) kf[t][s] = *(const f32x4 *)(Ks + (key0 + 16 * t + i) * P + 32 * h + 16 * s + 4 * g);
    float vf[KT][4][2];
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) vf[t][e][dt] = Vs[(key0 + 16 * t + 4 * g + e) * P + 32 * h + 16 * dt + i];
#pragma unroll
    for (int t = 0; t < KT; ++t) st[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < KT; ++t) st[t] = mfma_f32(kf[t][s][e], qf[s][e], st[t]);
    // softmax (Eq. 1)
    float m = -3.0e38f;                                   // a half without keys weighs nothing
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (key0 + 16 * t + 4 * g + j >= kn) st[t][j] = -INFINITY;
            m = fmaxf(m, st[t][j]);
        }
    m = cross_row_max(m);
    float l = 0.f;
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            st[t][j] = __builtin_amdgcn_exp2f(st[t][j] - m);
            l += st[t][j];
        }
    l = cross_row_sum(l);
    // O^T[channel 16 dt + 4 g + j][query i] += V^T P^T
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) acc[dt] = mfma_f32(vf[t][e][dt], st[t][e], acc[dt]);
    if (HALVES == 1) {
        const float inv = 1.0f / l;
        acc[0] *= inv;
        acc[1] *= inv;
    } else if (g == 0) {
        state[(half * HEADS + h) * 16 + i] = f32x2{m, l};
    }
    // Q has been read by all wavefronts before the barrier above
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) *(f32x4 *)(Qs + (16 * half + i) * P + 32 * h + 16 * dt + 4 * g) = acc[dt];
    __syncthreads();
    // Y = (O + LCE) Wo (Eq. 2)
    f32x4 oa[C / 16];
#pragma unroll
    for (int s = 0; s < C / 16; ++s) {
        const float *o = Qs + i * P + 16 * s + 4 * g;
        const f32x4 lce = *(const f32x4 *)(Ls + i * P + 16 * s + 4 * g);
        if (HALVES == 1) {
            oa[s] = *(const f32x4 *)o + lce;
        } else {
            const f32x2 a0 = state[(s / 2) * 16 + i], a1 = state[(HEADS + s / 2) * 16 + i];
            const float top = fmaxf(a0[0], a1[0]), f0 = __builtin_amdgcn_exp2f(a0[0] - top), f1 = __builtin_amdgcn_exp2f(a1[0] - top);
            const float inv = 1.0f / fmaf(a0[1], f0, a1[1] * f1);
            oa[s] = *(const f32x4 *)o * (f0 * inv) + *(const f32x4 *)(o + 16 * P) * (f1 * inv) + lce;
        }
    }
#pragma unroll
    for (int u = 0; u < NOT; ++u) {
        f32x4 out = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < C / 16; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) out = mfma_f32(oa[s][e], wo[u][s][e], out);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            Y[(img + region_token(D, r, 4 * g + j)) * C + 16 * (wave + 4 * u) + i] = out[j];
    }
}

template <typename K>
bool opt_in(K kernel, size_t bytes, bool &done)
{
    if (done || bytes <= 64 * 1024) return true;
    if (hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
        return false;
    done = true;
    return true;
}

template <int C>
int forward_c(const Dims &D, const float *X, const float *Wqkv, const float *Wo, const float *Wlce, float *Y,
              int32_t *Ir_out_opt, const int32_t *Ir_in_opt, float *qkv, float *pq, float *pk, hipStream_t st)
{
    static bool opted = false;
    if (!opt_in(k_f32_attn<C>, F32Smem<C>::bytes, opted)) return BRA_ERR_LAUNCH;
    {
        ProfScope ps(st, K_GEN_GEMM_QKV);
        hipLaunchKernelGGL((k_f32_qkv<C, false>), dim3(D.B * D.R), dim3(256), 0, st, X, Wqkv, qkv, pq, pk, D);
    }
    {
        ProfScope ps(st, K_GEN_ATTENTION);
        hipLaunchKernelGGL(k_f32_attn<C>, dim3(D.B * D.R), dim3(256), F32Smem<C>::bytes, st, qkv, pq, pk, Ir_in_opt,
                           Ir_out_opt, Wlce, Wo, Y, D);
    }
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

template <int C>
int route_c(const Dims &D, const float *X, const float *Wqkv, int32_t *Ir, float *Ar_opt, float *qkv, float *pq,
            float *pk, hipStream_t st)
{
    {
        ProfScope ps(st, K_GEN_GEMM_QKV);
        hipLaunchKernelGGL((k_f32_qkv<C, true>), dim3(D.B * D.R), dim3(256), 0, st, X, Wqkv, qkv, pq, pk, D);
    }
    {
        ProfScope ps(st, K_GEN_TOPK);
        hipLaunchKernelGGL(k_f32_route<C>, dim3(D.B * D.R), dim3(256), 0, st, pq, pk, Ir, Ar_opt, D);
    }
    return hipGetLastError() == hipSuccess ? BRA_OK : BRA_ERR_LAUNCH;
}

}  // namespace

// As long as the workgroups (image, region) run about at once, one per compute unit with 128 channels and two with 64, which take so
// little time that two rounds and a half are still faster than the general kernels' launches.  Here / there (us, regions of 4 x 4 tokens, 49
// per image, k = 4): C = 128: 4 images 20.6 / 33, 6 35.7 / 35.4, 10 38.9 / 37.6, 16 64.5 / 52.9; C = 64: 1 image 9.7 / 25, 24 33.9 / 41.8, 32 41.1 /
// 43.7, bra_route 14.7 / 13.7 (13.8 with the general kernels' own means), 64 67.5 / 72.7, bra_route 23.2 / 16.1.
bool f32_small_ok(const Dims &D)
{
    static const bool off = experiment_flag("BRA_NO_F32_SMALL");
    return !off && D.dtype == BRA_F32 && D.rh == 4 && D.rw == 4 && D.d == 32 && (D.C == 64 || D.C == 128) &&
           D.R <= 64 && D.k * kN <= kKeys && (long)D.B * D.R <= (D.C == 64 ? 1400 : 256);
}

int f32_small_forward(const Dims &D, const float *X, const float *Wqkv, const float *Wo, const float *Wlce, float *Y,
                      int32_t *Ir_out_opt, const int32_t *Ir_in_opt, float *qkv, float *pq, float *pk, hipStream_t st)
{
    if (D.C == 64) return forward_c<64>(D, X, Wqkv, Wo, Wlce, Y, Ir_out_opt, Ir_in_opt, qkv, pq, pk, st);
    return forward_c<128>(D, X, Wqkv, Wo, Wlce, Y, Ir_out_opt, Ir_in_opt, qkv, pq, pk, st);
}

int f32_small_route(const Dims &D, const float *X, const float *Wqkv, int32_t *Ir, float *Ar_opt, float *qkv,
                    float *pq, float *pk, hipStream_t st)
{
    if (D.C == 64) return route_c<64>(D, X, Wqkv, Ir, Ar_opt, qkv, pq, pk, st);
    return route_c<128>(D, X, Wqkv, Ir, Ar_opt, qkv, pq, pk, st);
}

}  // namespace bra
