// su2_learned.hip -- gfx950 kernels that train the learned a0 proposal.
//
// The network maps f(alpha) (log-scaled alpha in [0.5, 30]) through an MLP
// 1 -> 32 -> 32 -> 47 (tanh, tanh, linear) to the 47 parameters of a 16-bin
// monotone rational-quadratic spline g on [-1, 1] (Durkan et al. 2019; widths
// and heights 2 (m + (1 - 16 m) softmax), m = 1e-3; interior derivatives
// 1e-3 + softplus, boundary derivatives 1).  The proposal density of a0 is
// q(a0 | alpha) = g'(a0) / 2.  Training minimises the negative
// log-likelihood of exact heat-bath draws (Sec. 2 density of a0) with Adam:
//   data       one thread per sample: alpha log-uniform, a0 exact sampler
//   step       one wave per 16 samples: forward, analytic backward and the
//              weight gradient, summed over the workgroup
//   reduce     the workgroups' sums in a fixed order, then Adam
// Every sum has a fixed order, so training is bit-reproducible.
#include "su2_internal.h"

using namespace su2dev;

namespace su2rt {

namespace {

constexpr int OFF_W1 = 0, OFF_B1 = 32, OFF_W2 = 64, OFF_B2 = 1088, OFF_W3 = 1120,
              OFF_B3 = 2624;
constexpr int NBINS = 16;
constexpr float MIN_BIN = 1e-3f, MIN_DERIV = 1e-3f;

__device__ __forceinline__ float nn_feature(float alpha)
{
    return 2.0f * __log2f(alpha / kNNAlphaLo) / kNNLog2Range - 1.0f;
}

__device__ __forceinline__ float softplusf(float t) { return t > 20.0f ? t : log1pf(expf(t)); }
__device__ __forceinline__ float sigmoidf(float t) { return 1.0f / (1.0f + expf(-t)); }

// MLP forward from parameters P (global or LDS).
__device__ __forceinline__ void mlp_forward(const float *P, float f, float h1[32], float h2[32],
                                            float o[47])
{
#pragma unroll
    for (int j = 0; j < 32; ++j) h1[j] = tanhf(P[OFF_W1 + j] * f + P[OFF_B1 + j]);
    for (int j = 0; j < 32; ++j) {
        float a = P[OFF_B2 + j];
#pragma unroll
        for (int m = 0; m < 32; ++m) a += P[OFF_W2 + j * 32 + m] * h1[m];
        h2[j] = tanhf(a);
    }
    for (int i = 0; i < 47; ++i) {
        float a = P[OFF_B3 + i];
#pragma unroll
        for (int m = 0; m < 32; ++m) a += P[OFF_W3 + i * 32 + m] * h2[m];
        o[i] = a;
    }
}

// Softmax of 16 logits into bin sizes 2 (m + (1 - 16 m) p); p returned too.
__device__ __forceinline__ void bin_sizes(const float *logit, float p[16], float sz[16])
{
    float mx = logit[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, logit[i]);
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum += (p[i] = expf(logit[i] - mx));
    const float inv = 1.0f / sum;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        p[i] *= inv;
        sz[i] = 2.0f * (MIN_BIN + (1.0f - NBINS * MIN_BIN) * p[i]);
    }
}

// ------------------------------------------------------------------- data
__global__ void nn_data_kernel(float *__restrict__ alpha, float *__restrict__ a0, int64_t n,
                               float lo, float log2ratio, uint32_t k0, uint32_t k1)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t site = (uint32_t)i;
    const U4 wa = philox(site, 0u, word2(0u, TAG_TRAIN, 0u), 0u, k0, k1);
    const float al = lo * exp2f(u01(wa.a) * log2ratio);
    const uint32_t w2 = word2(1u, TAG_TRAIN, 0u);
    const U4 w0 = philox(site, 0u, w2, 0u, k0, k1);
    alpha[i] = al;
    a0[i] = 1.0f - sample_delta(al, w0, site, 0u, w2, k0, k1);
}

// ------------------------------------------------------------ training step
// One launch takes a minibatch through the network, the spline and back, and
// leaves the gradient as one FP64 partial sum per workgroup; nn_reduce_kernel
// adds the partials and takes the Adam step.
//
// A wave works on 16 samples at a time and needs no other wave until its sums
// are complete.  The four matrix products of the MLP (W2 h1, W3 h2, W3^T do,
// W2^T dz2) are v_mfma_f32_16x16x4 over [neuron][sample] tiles with the inner
// index in increasing order, whose result is the chain of FP32 FMAs in that
// order, bit for bit; activations pass through LDS between them (11.5 KB a
// wave) because the next product and the weight gradient index them the other
// way round.  The spline of a sample is shared by its four lanes: lanes of
// even 16-lane groups hold the widths, odd ones the heights.  The gradients are
// FP32 products summed in FP64, one sum per lane: the workgroup's 64 samples
// for W2 and W3 (8 sums a lane), the wave's 16 for the rest.
//
// Bound: a batch of 16384 is one wave per SIMD and 32 thousand cycles of
// dependent work in it, a third of them the conversions of the gradient's FP32
// products to FP64 (v_cvt_f64_f32, about 15 cycles a wave; an FP64 MFMA would
// take the products unrounded, six times cheaper, but to other bits).  Nothing
// of the per-sample record goes to memory.  Measured per Adam step of 16384
// samples: 23.5 us (this kernel 17, the reduction 4, the rest launch gaps)
// against 139 us with one thread per sample, its record in memory and one
// workgroup per parameter summing it (77 + 43 + 16 + 5 us); the same bits.
// LDS strides of a row of 32 and of 48 values: 16-byte rows, and the 16 rows x 4
// consecutive columns that an MFMA operand reads fall on 64 different banks
constexpr int HS = 36, OS = 52;
constexpr int LW1 = 0, LB1 = 32, LW2 = 64, LB2 = LW2 + 32 * HS, LW3 = LB2 + 32,
              LB3 = LW3 + 48 * HS, LPARAMS = LB3 + 48;  // LDS copy of the parameters
constexpr int WH1 = 0, WH2 = 16 * HS, WD1 = 32 * HS, WD2 = 48 * HS, WDO = 64 * HS,
              WF = WDO + 16 * OS, WK = WF + 16, WLDS = WK + 16;  // per-wave LDS (floats)
constexpr int NNWAVES = kNNTile / 16;

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Orders the LDS accesses of a wave's lanes: the LDS serves a wave's
// instructions in order, so the compiler is all that has to be held.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// loss_b = -(ln 1/2 + ln g'(a0)); part[workgroup][p] = the workgroup's sum of
// d(mean loss)/d(param p), p = kNNParams its sum of losses.
__global__ __launch_bounds__(256, 2) void nn_step_kernel(const float *__restrict__ params,
                                                         const float *__restrict__ alpha,
                                                         const float *__restrict__ a0,
                                                         int64_t offset, int batch, int64_t n,
                                                         double *__restrict__ part,
                                                         float inv_batch)
{
    __shared__ float P[LPARAMS];
    __shared__ __align__(16) float act[NNWAVES * WLDS];
    __shared__ double gder[NNWAVES * 15 * 32];  // derivative rows of W3, per wave
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int j = lane & 15, q = lane >> 4;  // sample of the tile; 16-lane group
    // the sample of this lane at a tile (a lane without one takes the batch's first)
    auto at = [&](int base) {
        const int b = base + 16 * wv + j;
        int64_t i = offset + (b < batch ? b : 0);
        if (i >= n) {  // offset < n, so one subtraction unless the batch wraps twice
            i -= n;
            if (i >= n) i %= n;
        }
        return i;
    };
    int64_t idx = at((int)blockIdx.x * kNNTile);
    float al = alpha[idx], x0 = a0[idx];
    {
        // all loads first: one round trip to memory instead of one per 256 parameters
        constexpr int NP = (kNNParams + 255) / 256;
        float v[NP];
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int i = (int)threadIdx.x + 256 * u;
            v[u] = i < kNNParams ? params[i] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int i = (int)threadIdx.x + 256 * u;
            int d = i;  // W1, b1
            if (i >= OFF_B3) d = LB3 + i - OFF_B3;
            else if (i >= OFF_W3) d = LW3 + ((i - OFF_W3) >> 5) * HS + ((i - OFF_W3) & 31);
            else if (i >= OFF_B2) d = LB2 + i - OFF_B2;
            else if (i >= OFF_W2) d = LW2 + ((i - OFF_W2) >> 5) * HS + ((i - OFF_W2) & 31);
            if (i < kNNParams) P[d] = v[u];
        }
    }
    if (threadIdx.x < 32) P[LW3 + 47 * HS + threadIdx.x] = 0.0f;  // padding row of outputs
    if (threadIdx.x == 32) P[LB3 + 47] = 0.0f;
    __syncthreads();
    float *const L = act + wv * WLDS;
    float *const H1 = L + WH1, *const H2 = L + WH2, *const D1 = L + WD1, *const D2 = L + WD2,
                *const DO = L + WDO, *const F = L + WF;
    int *const KB = reinterpret_cast<int *>(L + WK);
    // weight gradients over the workgroup's 64 samples: group grp of 32 lanes
    // holds column m0 of rows 4 grp + r of W3 (widths and heights) and of W2
    const int m0 = lane & 31, half = lane >> 5, grp = 2 * wv + half;
    double g3[4] = {0.0, 0.0, 0.0, 0.0}, g2[4] = {0.0, 0.0, 0.0, 0.0};
    // over the wave's own 16 samples, lane i: b3[i]; b2[i] (i < 32) or b1[i - 32];
    // W1[i - 32] (i >= 32); loss
    double gb3 = 0.0, gb = 0.0, gw1 = 0.0, gloss = 0.0;
    double *const GD = gder + wv * 15 * 32;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (64 * i + lane < 15 * 32) GD[64 * i + lane] = 0.0;
    for (int base = (int)blockIdx.x * kNNTile; base < batch; base += (int)gridDim.x * kNNTile) {
        const int b = base + 16 * wv + j;
        const bool live = b < batch, ragged = batch - base < kNNTile;  // (uniform)
        // A lane without a sample repeats the batch's first one, with zero in place
        // of its gradients: a product with them is zero, or the NaN that the sample
        // itself gives
        const float f = nn_feature(al), xv = x0;
        const int next = base + (int)gridDim.x * kNNTile;
        if (next < batch) {
            idx = at(next);
            al = alpha[idx];
            x0 = a0[idx];
        }
        // layer 1, in the B operand's layout (inner index 4 kk + q)
        float h[8];
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const int m = 4 * kk + q;
            h[kk] = tanhf(P[LW1 + m] * f + P[LB1 + m]);
            H1[j * HS + m] = h[kk];
        }
        if (q == 0) F[j] = f;
        // layer 2
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x4 c;
#pragma unroll
            for (int v = 0; v < 4; ++v) c[v] = P[LB2 + 16 * t + 4 * q + v];
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(P[LW2 + (16 * t + j) * HS + 4 * kk + q],
                                                         h[kk], c, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) H2[j * HS + 16 * t + 4 * q + v] = tanhf(c[v]);
        }
        wave_sync();
        // layer 3 (47 outputs and a zero row)
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) h[kk] = H2[j * HS + 4 * kk + q];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            f32x4 c;
#pragma unroll
            for (int v = 0; v < 4; ++v) c[v] = P[LB3 + 16 * t + 4 * q + v];
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(P[LW3 + (16 * t + j) * HS + 4 * kk + q],
                                                         h[kk], c, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) DO[j * OS + 16 * t + 4 * q + v] = c[v];
        }
        wave_sync();
        // spline: this lane's 16 logits are the widths (even q) or the heights
        const int hpart = q & 1;
        float lg[16], p[16], sz[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) lg[i] = DO[j * OS + 16 * hpart + i];
        bin_sizes(lg, p, sz);
        // bin k of xv and its left knot x_k (cumulative widths, from the width lanes)
        int k = 0;
        float xk = -1.0f, cum = -1.0f;
#pragma unroll
        for (int i = 0; i < 15; ++i) {
            cum += sz[i];
            if (xv >= cum) {
                k = i + 1;
                xk = cum;
            }
        }
        k = __shfl(k, j, 64);
        xk = __shfl(xk, j, 64);
        float szk = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) szk = i == k ? sz[i] : szk;
        float Wk = __shfl(szk, j, 64);
        const float Hk = __shfl(szk, j + 16, 64);
        // interior derivatives d_i = 1e-3 + softplus(o[31 + i]), i = 1..15; the ends are 1
        float thl = 0.0f, thh = 0.0f, dl = 1.0f, dh = 1.0f;
        if (k > 0) {
            thl = DO[j * OS + 31 + k];
            dl = MIN_DERIV + softplusf(thl);
        }
        if (k < NBINS - 1) {
            thh = DO[j * OS + 32 + k];
            dh = MIN_DERIV + softplusf(thh);
        }
        if (k == NBINS - 1) Wk = 1.0f - xk;  // last knot is exactly 1
        const float s = Hk / Wk;
        const float xi = (xv - xk) / Wk;
        const float om = xi * (1.0f - xi);
        const float tt = dh + dl - 2.0f * s;
        const float den = s + tt * om;
        const float num = dh * xi * xi + 2.0f * s * om + dl * (1.0f - xi) * (1.0f - xi);
        const float ell = 2.0f * logf(s) + logf(num) - 2.0f * logf(den);
        const bool undefined = __any(ell != ell);  // (uniform)
        if (live && q == 0) gloss += (double)-(-0.69314718055994531f + ell);

        // d ell / d(s, xi, d_k, d_k+1)
        const float dN_ds = 2.0f * om, dD_ds = 1.0f - 2.0f * om;
        const float dN_dxi =
            2.0f * dh * xi + 2.0f * s * (1.0f - 2.0f * xi) - 2.0f * dl * (1.0f - xi);
        const float dD_dxi = tt * (1.0f - 2.0f * xi);
        const float inum = 1.0f / num, iden = 1.0f / den;
        const float l_s = 2.0f / s + dN_ds * inum - 2.0f * dD_ds * iden;
        const float l_xi = dN_dxi * inum - 2.0f * dD_dxi * iden;
        const float l_dl = (1.0f - xi) * (1.0f - xi) * inum - 2.0f * om * iden;
        const float l_dh = xi * xi * inum - 2.0f * om * iden;
        // chain to the bin width, height and left knot
        const float l_H = l_s / Wk;
        const float l_W = -(l_s * s + l_xi * xi) / Wk;
        const float l_x = -l_xi / Wk;
        // widths: g_i = [i == k] l_W + [i < k] l_x; heights: g_i = [i == k] l_H
        // softmax backward: d/dtheta_m = 2 (1 - 16 m) p_m (g_m - sum_i p_i g_i)
        const float gk = hpart ? l_H : l_W, glt = hpart ? 0.0f : l_x;
        float sp = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float g = (i == k ? gk : 0.0f) + (i < k ? glt : 0.0f);
            sp += p[i] * g;
        }
        const float cs = 2.0f * (1.0f - NBINS * MIN_BIN);
        // the mean loss is -ell / batch per sample: scale = -inv_batch
        const float sc = -inv_batch;
        float dlo = 0.0f, dhi = 0.0f;
        if (k > 0) dlo = l_dl * sigmoidf(thl);
        if (k < NBINS - 1) dhi = l_dh * sigmoidf(thh);
        wave_sync();  // every lane has read its outputs; they are replaced by their gradients
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float g = (i == k ? gk : 0.0f) + (i < k ? glt : 0.0f);
            const float d = sc * cs * p[i] * (g - sp);
            // the two lanes that hold the same half write eight entries each
            if ((i >> 3) == (q >> 1)) DO[j * OS + 16 * hpart + i] = live ? d : 0.0f;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 4 * q + v;  // derivative i + 1; entry 15 is the padding column
            float g = 0.0f;
            if (i + 1 == k) g = dlo;
            if (i == k && i < NBINS - 1) g = dhi;
            DO[j * OS + 32 + i] = live ? sc * g : 0.0f;
        }
        wave_sync();
        // back through layer 3: dz2 = (W3^T do) (1 - h2^2)
        float d[12];
#pragma unroll
        for (int kk = 0; kk < 12; ++kk) d[kk] = DO[j * OS + 4 * kk + q];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x4 c{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kk = 0; kk < 12; ++kk)
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(P[LW3 + (4 * kk + q) * HS + 16 * t + j],
                                                         d[kk], c, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = 16 * t + 4 * q + v;
                const float hm = H2[j * HS + m], a = c[v];
                D2[j * HS + m] = a * (1.0f - hm * hm);
            }
        }
        if (ragged && !live)
            for (int v = 0; v < 8; ++v) D2[j * HS + 16 * (v >> 2) + 4 * q + (v & 3)] = 0.0f;
        wave_sync();
        // back through layer 2: dz1 = (W2^T dz2) (1 - h1^2)
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) h[kk] = D2[j * HS + 4 * kk + q];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x4 c{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(P[LW2 + (4 * kk + q) * HS + 16 * t + j],
                                                         h[kk], c, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = 16 * t + 4 * q + v;
                const float hm = H1[j * HS + m], a = c[v];
                D1[j * HS + m] = a * (1.0f - hm * hm);
            }
        }
        if (ragged && !live)
            for (int v = 0; v < 8; ++v) D1[j * HS + 16 * (v >> 2) + 4 * q + (v & 3)] = 0.0f;
        if (q == 0) KB[j] = k;
        wave_sync();
        // biases and W1, one sample after the other: FP32 products, FP64 sums.  Of the
        // 15 derivative rows of W3 a sample touches the two at its bin's ends:
        // the lower half of the wave adds row k - 1, the upper half row k, to
        // sums in LDS (in sample order: the LDS serves a wave's adds in turn).  The
        // other rows' products are zero times an activation: nothing but for a NaN,
        // which shows in the sample's loss
        const int o3 = lane < 47 ? lane : 47;
        const float *const db = half ? D1 + m0 : D2 + m0;
        int row[16];
        float pr[16];
#pragma unroll
        for (int sm = 0; sm < 16; ++sm) {
            row[sm] = KB[sm] - 1 + half;
            pr[sm] = H2[sm * HS + m0];
        }
#pragma unroll
        for (int sm = 0; sm < 16; ++sm) {
            gb3 += (double)DO[sm * OS + o3];
            const float z = db[sm * HS];
            gb += (double)z;
            gw1 += (double)(z * F[sm]);  // W1 in the upper lanes (the lower ones' is unused)
            // a row outside 0..14 reads inside the sample's record and is not added
            pr[sm] *= DO[sm * OS + 32 + row[sm]];
        }
        if (undefined && half == 0) {
            float nil = 0.0f;
            for (int sm = 0; sm < 16; ++sm) nil += H2[sm * HS + m0] * 0.0f;
            for (int r = 0; r < 15; ++r) GD[r * 32 + m0] += (double)nil;
        }
#pragma unroll
        for (int sm = 0; sm < 16; ++sm)
            if ((unsigned)row[sm] < 15u)
                __hip_atomic_fetch_add(GD + row[sm] * 32 + m0, (double)pr[sm], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
#pragma unroll 4
        for (int sm = 0; sm < kNNTile; ++sm) {
            const float *const S = act + (sm >> 4) * WLDS;
            const int i = sm & 15;
            const float x = S[WH2 + i * HS + m0], y = S[WH1 + i * HS + m0];
            const float4 a = *reinterpret_cast<const float4 *>(S + WDO + i * OS + 4 * grp);
            const float4 z = *reinterpret_cast<const float4 *>(S + WD2 + i * HS + 4 * grp);
            g3[0] += (double)(a.x * x);
            g3[1] += (double)(a.y * x);
            g3[2] += (double)(a.z * x);
            g3[3] += (double)(a.w * x);
            g2[0] += (double)(z.x * y);
            g2[1] += (double)(z.y * y);
            g2[2] += (double)(z.z * y);
            g2[3] += (double)(z.w * y);
        }
        __syncthreads();  // the next tile overwrites the activations
    }
    double *const out = part + (size_t)blockIdx.x * kNNPart;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        out[OFF_W3 + (4 * grp + r) * 32 + m0] = g3[r];
        out[OFF_W2 + (4 * grp + r) * 32 + m0] = g2[r];
    }
    // the four waves' other sums, added in wave order through LDS
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) gloss += __shfl_down(gloss, off, 64);
    double *const red = reinterpret_cast<double *>(act) + wv * 4 * 64 + lane;
    red[0] = gb3;
    red[64] = gb;
    red[128] = gw1;
    red[192] = gloss;
    __syncthreads();
    for (int i = threadIdx.x; i < 15 * 32; i += blockDim.x) {
        double t = gder[i];
#pragma unroll
        for (int w = 1; w < NNWAVES; ++w) t += gder[w * 15 * 32 + i];
        out[OFF_W3 + 32 * 32 + i] = t;
    }
    double t = reinterpret_cast<double *>(act)[threadIdx.x];
#pragma unroll
    for (int w = 1; w < NNWAVES; ++w) t += reinterpret_cast<double *>(act)[w * 4 * 64 + threadIdx.x];
    if (wv == 0 && lane < 47) out[OFF_B3 + lane] = t;
    if (wv == 1) out[lane < 32 ? OFF_B2 + lane : OFF_B1 + lane - 32] = t;
    if (wv == 2 && lane >= 32) out[OFF_W1 + lane - 32] = t;
    if (wv == 3 && lane == 0) out[kNNParams] = t;
}

// Adam (Kingma & Ba 2015) with bias corrections bc1 = 1 - b1^t, bc2 = 1 - b2^t.
struct Adam {
    float lr, b1, b2, eps, bc1, bc2;
};

// Sum of the workgroups' partials in a fixed order: 16 parameters per
// workgroup (one 128-byte line of a partial), slice s of 16 adds partials s,
// s + 16, ... in turn, then the slices are added in order.  The gradient is
// stored; with `step` the parameter takes its Adam step; entry kNNParams is
// the mean loss.
constexpr int RP = 16, RS = 16;
__global__ __launch_bounds__(RP *RS) void nn_reduce_kernel(const double *__restrict__ part,
                                                           int npart, int batch,
                                                           float *__restrict__ grad,
                                                           double *__restrict__ loss_out, int step,
                                                           float *__restrict__ params,
                                                           float *__restrict__ m,
                                                           float *__restrict__ v, Adam o)
{
    __shared__ double sum[RS][RP];
    const int c = threadIdx.x % RP, s = threadIdx.x / RP;
    const int p = (int)blockIdx.x * RP + c;
    double t = 0.0;
    if (p <= kNNParams) {
#pragma unroll 16
        for (int w = s; w < npart; w += RS) t += part[(size_t)w * kNNPart + p];
    }
    sum[s][c] = t;
    __syncthreads();
    if (s != 0 || p > kNNParams) return;
#pragma unroll
    for (int i = 1; i < RS; ++i) t += sum[i][c];
    if (p == kNNParams) {
        if (loss_out) *loss_out = t / batch;
        return;
    }
    const float g = (float)t;
    grad[p] = g;
    if (!step) return;
    const float mi = o.b1 * m[p] + (1.0f - o.b1) * g;
    const float vi = o.b2 * v[p] + (1.0f - o.b2) * g * g;
    m[p] = mi;
    v[p] = vi;
    params[p] -= o.lr * (mi / o.bc1) / (sqrtf(vi / o.bc2) + o.eps);
}

// One thread per table row: rows at f = -1 + 2 j / 255.
__global__ void nn_table_kernel(const float *__restrict__ params, float *__restrict__ table)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= kNNRows) return;
    const float f = -1.0f + 2.0f * (float)j / (float)(kNNRows - 1);
    float h1[32], h2[32], o[47];
    mlp_forward(params, f, h1, h2, o);
    float p[16], sz[16];
    float *row = table + (size_t)j * kNNRow;
    for (int part = 0; part < 2; ++part) {
        bin_sizes(o + 16 * part, p, sz);
        float c = -1.0f;
        for (int i = 0; i < 15; ++i) {
            c += sz[i];
            row[16 * part + i] = c;
        }
        row[16 * part + 15] = 1.0f;
    }
    for (int i = 0; i < 15; ++i) row[32 + i] = MIN_DERIV + softplusf(o[32 + i]);
    row[47] = 1.0f;
}

__global__ void test_learned_kernel(const float *__restrict__ table, const float4 *__restrict__ V,
                                    const float4 *__restrict__ Uold, int64_t n, float beta,
                                    uint32_t k0, uint32_t k1, uint32_t sweep, uint32_t mu,
                                    uint32_t replica, float orw, float4 *__restrict__ out,
                                    int32_t *__restrict__ accepted)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float4 v = V[i], u = Uold[i];
    int acc = 0;
    const Q r = learned_link(Q{v.x, v.y, v.z, v.w}, Q{u.x, u.y, u.z, u.w}, table, beta,
                             (uint32_t)i, sweep, mu, replica, k0, k1, acc, orw);
    out[i] = make_float4(r.w, r.x, r.y, r.z);
    if (accepted) accepted[i] = acc;
}

inline unsigned nblk(uint64_t n, unsigned b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

hipError_t launch_nn_data(float *alpha, float *a0, int64_t n, float lo, float hi, uint64_t seed,
                          hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(nn_data_kernel, dim3(nblk((uint64_t)n, 256)), dim3(256), 0, stream, alpha,
                       a0, n, lo, log2f(hi / lo), (uint32_t)seed, (uint32_t)(seed >> 32));
    return hipGetLastError();
}

hipError_t launch_nn_step(const NNBuffers &nb, int64_t offset, int batch, int64_t n,
                          double *loss_out, float lr, int step, hipStream_t stream)
{
    const int wg = nn_parts(batch);
    hipLaunchKernelGGL(nn_step_kernel, dim3(wg), dim3(64 * NNWAVES), 0, stream, nb.params, nb.alpha,
                       nb.a0, offset, batch, n, nb.part, 1.0f / (float)batch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const float b1 = 0.9f, b2 = 0.999f;
    const Adam o{lr, b1, b2, 1e-8f, 1.0f - powf(b1, (float)step), 1.0f - powf(b2, (float)step)};
    hipLaunchKernelGGL(nn_reduce_kernel, dim3(nblk(kNNPart, RP)), dim3(RP * RS), 0, stream,
                       nb.part, wg, batch, nb.grad, loss_out, step, nb.params, nb.m, nb.v, o);
    return hipGetLastError();
}

hipError_t launch_nn_table(const float *params, float *table, hipStream_t stream)
{
    hipLaunchKernelGGL(nn_table_kernel, dim3(1), dim3(kNNRows), 0, stream, params, table);
    return hipGetLastError();
}

hipError_t launch_test_learned(const float *table, const float *V, const float *Uold, int64_t n,
                               float beta, uint64_t seed, uint32_t sweep, uint32_t mu,
                               uint32_t replica, float orw, float *out, int32_t *accepted,
                               hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(test_learned_kernel, dim3(nblk((uint64_t)n, 256)), dim3(256), 0, stream,
                       table, (const float4 *)V, (const float4 *)Uold, n, beta, (uint32_t)seed,
                       (uint32_t)(seed >> 32), sweep, mu, replica, orw, (float4 *)out, accepted);
    return hipGetLastError();
}

}  // namespace su2rt
