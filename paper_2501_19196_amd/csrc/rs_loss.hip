// Training loss of one image against its target and its gradient
// (Sec. 3, loss function; App. A.7): per colour channel
//   L_ch = (1 - lambda) mean (I - I^)^2 + lambda (1 - mean SSIM) / 2,
// averaged over the three channels. SSIM uses window moments of a normalised
// Gaussian window (zero outside the image); the gradient of mean SSIM is
// App. A.7's (1/hw) ((E * w) + I^ (F * w) - I (G * w)).
//
// Three launches: k_ssim_maps (window moments, the SSIM map and the squared error summed per workgroup,
// the E, F, G maps written), k_ssim_grad (window sums of E, F, G, then the per-pixel gradient) and
// k_loss_total.
#include <math.h>

#include <mutex>

#include "rs_internal.h"

namespace rs {

// The window sums run down the image: a wave owns 64 columns of an image row taken as 3 w floats (pixel
// and channel alike: a tap is 3 floats apart) and a band of rows. For each input row it puts the row's
// values in LDS, a lane sums them across, and adds the sums to the output rows that they belong to, whose
// partial sums stay in registers (a ring of 2 R + 1, in code unrolled over its phases). So a row is read
// once per band, no barrier is needed, and each sum is taken in the order of the taps. Bound by vector
// arithmetic: about 180 operations per channel of a pixel in k_ssim_maps and 90 in k_ssim_grad.
// 1920x1080, loss and gradient: 98 us; 228 us with LDS tiles of 32x8 and vertical sums taken tap by tap from LDS.
constexpr int kLossWaves = 4;                 // waves of a workgroup, side by side
constexpr int kLossCols = kLossWaves * 64;    // columns of a workgroup
constexpr int kMaxRadius = 7;
constexpr int kLossFill = 256;  // workgroups a launch should have at least, one per CU (800x800: 51 us, 55 at 512)

struct LossConst {
    int64_t cols;                // 3 w
    int32_t w, h, band, strips;  // rows per band; workgroups across
    int32_t want_grad;
    float lambda;
    float g[2 * kMaxRadius + 1];  // normalised 1-D window (the 2-D window is its outer product)
};

// orders a wave's LDS accesses (its own lanes' stores before its loads, and those before the next stores)
__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(R > 6 ? 3 : 4))) void k_ssim_maps(
    const float *__restrict__ img, const float *__restrict__ tgt, float *__restrict__ efg, float *__restrict__ partial,
    const LossConst L)
{
    constexpr int W = 2 * R + 1, Line = 64 + 6 * R;
    __shared__ float4 line4[kLossWaves][Line];  // I, I^, I^2, I^^2
    __shared__ float line1[kLossWaves][Line];   // I I^
    __shared__ double red[kLossWaves][6];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c0 = int64_t(blockIdx.x % L.strips) * kLossCols + wave * 64;
    const int y0 = (blockIdx.x / L.strips) * L.band;
    const int rows = min(L.band, L.h - y0);
    const int64_t c = c0 + lane;
    // the line's columns c0 - 3 R + lane and, for the last 6 R, + 64; values outside the image are 0
    const int64_t ca = c0 - 3 * R + lane, cb = ca + 64;
    const bool in_a = ca >= 0 && ca < L.cols, in_b = lane < 6 * R && cb < L.cols && cb >= 0;
    const int64_t plane = L.cols * L.h;
    float acc[5][W], ci[W], ct[W];
    double ssim = 0.0, sq = 0.0;
    float ia = 0.0f, ta = 0.0f, ib = 0.0f, tb = 0.0f;
    auto fetch = [&](int i) {
        const int y = y0 - R + i;
        const bool in = y >= 0 && y < L.h;
        const int64_t at = int64_t(y) * L.cols;
        ia = in && in_a ? img[at + ca] : 0.0f;
        ta = in && in_a ? tgt[at + ca] : 0.0f;
        ib = in && in_b ? img[at + cb] : 0.0f;
        tb = in && in_b ? tgt[at + cb] : 0.0f;
    };
    const int n_in = rows + 2 * R;
    if (c0 < L.cols) {
        fetch(0);
        for (int base = 0; base < n_in; base += W) {
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const int i = base + k;
                if (i >= n_in) break;
                line4[wave][lane] = make_float4(ia, ta, ia * ia, ta * ta);
                line1[wave][lane] = ia * ta;
                if (lane < 6 * R) {
                    line4[wave][64 + lane] = make_float4(ib, tb, ib * ib, tb * tb);
                    line1[wave][64 + lane] = ib * tb;
                }
                fetch(i + 1 < n_in ? i + 1 : i);
                wave_lds_fence();
                float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f, s4 = 0.0f;
#pragma unroll
                for (int m = 0; m < W; ++m) {
                    const float4 v = line4[wave][lane + 3 * m];
                    const float p = line1[wave][lane + 3 * m];
                    if (m == R) {
                        ci[k] = v.x;
                        ct[k] = v.y;
                    }
                    s0 = __builtin_fmaf(L.g[m], v.x, s0);
                    s1 = __builtin_fmaf(L.g[m], v.y, s1);
                    s2 = __builtin_fmaf(L.g[m], v.z, s2);
                    s3 = __builtin_fmaf(L.g[m], v.w, s3);
                    s4 = __builtin_fmaf(L.g[m], p, s4);
                }
                wave_lds_fence();
#pragma unroll
                for (int m = 0; m < W; ++m) {
                    const int o = (k - m + W) % W;  // the output row that this row is tap m of
                    acc[0][o] = __builtin_fmaf(L.g[m], s0, m ? acc[0][o] : 0.0f);
                    acc[1][o] = __builtin_fmaf(L.g[m], s1, m ? acc[1][o] : 0.0f);
                    acc[2][o] = __builtin_fmaf(L.g[m], s2, m ? acc[2][o] : 0.0f);
                    acc[3][o] = __builtin_fmaf(L.g[m], s3, m ? acc[3][o] : 0.0f);
                    acc[4][o] = __builtin_fmaf(L.g[m], s4, m ? acc[4][o] : 0.0f);
                }
                if (i < 2 * R) continue;
                const int o = (k + 1) % W, centre = (k - R + W) % W;
                const float mu = acc[0][o], mh = acc[1][o], eaa = acc[2][o], ebb = acc[3][o], eab = acc[4][o];
                const float c1 = 1e-4f, c2 = 9e-4f;
                const float A = 2.0f * mu * mh + c1;
                const float B = 2.0f * (eab - mu * mh) + c2;
                const float C = mu * mu + mh * mh + c1;
                const float D = (eaa - mu * mu) + (ebb - mh * mh) + c2;
                const float inv = 1.0f / (C * D);
                const float S = A * B * inv;
                const float d = ci[centre] - ct[centre];
                if (c < L.cols) {
                    ssim += double(S);
                    sq += double(d * d);
                    if (L.want_grad) {
                        // App. A.7: E, F, G (factored through 1 / (C D) to stay in range)
                        const int64_t px = int64_t(y0 + i - 2 * R) * L.cols + c;
                        efg[px] = 2.0f * inv * (mh * (B - A) - S * mu * (D - C));
                        efg[plane + px] = 2.0f * A * inv;
                        efg[2 * plane + px] = 2.0f * S / D;
                    }
                }
            }
        }
    }
    // sums of the SSIM map and the squared error over the workgroup's columns and rows, per channel
    const int mine = int(c % 3);
    for (int ch = 0; ch < 3; ++ch) {
        double a = mine == ch ? ssim : 0.0, q = mine == ch ? sq : 0.0;
        for (int d = 32; d > 0; d >>= 1) {
            a += __shfl_xor(a, d);
            q += __shfl_xor(q, d);
        }
        if (lane == 0) {
            red[wave][ch] = a;
            red[wave][3 + ch] = q;
        }
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        double a = 0.0;
        for (int k = 0; k < kLossWaves; ++k) a += red[k][threadIdx.x];
        partial[6 * int64_t(blockIdx.x) + threadIdx.x] = float(a);
    }
}

template <int R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_ssim_grad(
    const float *__restrict__ img, const float *__restrict__ tgt, const float *__restrict__ efg, float *__restrict__ grad,
    const LossConst L)
{
    constexpr int W = 2 * R + 1, Line = 64 + 6 * R;
    __shared__ float2 line2[kLossWaves][Line];  // E, F
    __shared__ float line1[kLossWaves][Line];   // G
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c0 = int64_t(blockIdx.x % L.strips) * kLossCols + wave * 64;
    const int y0 = (blockIdx.x / L.strips) * L.band;
    if (c0 >= L.cols) return;
    const int rows = min(L.band, L.h - y0);
    const int64_t c = c0 + lane;
    const int64_t ca = c0 - 3 * R + lane, cb = ca + 64;
    const bool in_a = ca >= 0 && ca < L.cols, in_b = lane < 6 * R && cb < L.cols && cb >= 0;
    const int64_t plane = L.cols * L.h;
    const float inv_n = 1.0f / float(int64_t(L.w) * L.h);
    float acc[3][W];
    float ea = 0.0f, fa = 0.0f, ga = 0.0f, eb = 0.0f, fb = 0.0f, gb = 0.0f, I = 0.0f, T = 0.0f;
    auto fetch = [&](int i) {
        const int y = y0 - R + i;
        const bool in = y >= 0 && y < L.h;
        const int64_t at = int64_t(y) * L.cols;
        ea = in && in_a ? efg[at + ca] : 0.0f;
        fa = in && in_a ? efg[plane + at + ca] : 0.0f;
        ga = in && in_a ? efg[2 * plane + at + ca] : 0.0f;
        eb = in && in_b ? efg[at + cb] : 0.0f;
        fb = in && in_b ? efg[plane + at + cb] : 0.0f;
        gb = in && in_b ? efg[2 * plane + at + cb] : 0.0f;
        // the output row that this input row completes
        const bool out = i >= 2 * R && c < L.cols;
        const int64_t px = int64_t(y0 + i - 2 * R) * L.cols + c;
        I = out ? img[px] : 0.0f;
        T = out ? tgt[px] : 0.0f;
    };
    const int n_in = rows + 2 * R;
    fetch(0);
    for (int base = 0; base < n_in; base += W) {
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const int i = base + k;
            if (i >= n_in) break;
            line2[wave][lane] = make_float2(ea, fa);
            line1[wave][lane] = ga;
            if (lane < 6 * R) {
                line2[wave][64 + lane] = make_float2(eb, fb);
                line1[wave][64 + lane] = gb;
            }
            const float Io = I, To = T;
            fetch(i + 1 < n_in ? i + 1 : i);
            wave_lds_fence();
            float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;
#pragma unroll
            for (int m = 0; m < W; ++m) {
                const float2 v = line2[wave][lane + 3 * m];
                s0 = __builtin_fmaf(L.g[m], v.x, s0);
                s1 = __builtin_fmaf(L.g[m], v.y, s1);
                s2 = __builtin_fmaf(L.g[m], line1[wave][lane + 3 * m], s2);
            }
            wave_lds_fence();
#pragma unroll
            for (int m = 0; m < W; ++m) {
                const int o = (k - m + W) % W;
                acc[0][o] = __builtin_fmaf(L.g[m], s0, m ? acc[0][o] : 0.0f);
                acc[1][o] = __builtin_fmaf(L.g[m], s1, m ? acc[1][o] : 0.0f);
                acc[2][o] = __builtin_fmaf(L.g[m], s2, m ? acc[2][o] : 0.0f);
            }
            if (i < 2 * R || c >= L.cols) continue;
            const int o = (k + 1) % W;
            const float dssim = (acc[0][o] + To * acc[1][o] - Io * acc[2][o]) * inv_n;
            grad[int64_t(y0 + i - 2 * R) * L.cols + c] =
                (2.0f * (1.0f - L.lambda) * inv_n * (Io - To) - 0.5f * L.lambda * dssim) * (1.0f / 3.0f);
        }
    }
}

__global__ __launch_bounds__(256) void k_loss_total(const float *__restrict__ partial, int64_t n_tiles,
                                                    float *__restrict__ loss, const LossConst L)
{
    __shared__ double red[6][256];
    const int tid = threadIdx.x;
    double acc[6] = {0, 0, 0, 0, 0, 0};
    for (int64_t b = tid; b < n_tiles; b += 256)
        for (int k = 0; k < 6; ++k) acc[k] += double(partial[6 * b + k]);
    for (int k = 0; k < 6; ++k) red[k][tid] = acc[k];
    __syncthreads();
    for (int step = 128; step > 0; step >>= 1) {
        if (tid < step)
            for (int k = 0; k < 6; ++k) red[k][tid] += red[k][tid + step];
        __syncthreads();
    }
    if (tid == 0) {
        const double n = double(L.w) * double(L.h), lam = L.lambda;
        double tot = 0.0;
        for (int ch = 0; ch < 3; ++ch)
            tot += (1.0 - lam) * red[3 + ch][0] / n + lam * (1.0 - red[ch][0] / n) * 0.5;
        loss[0] = float(tot / 3.0);
    }
}

// ------------------------------------------------------------------- host

static LossConst loss_const(int32_t w, int32_t h, const rs_loss_params *lp, bool grad)
{
    const int r = lp->radius;
    LossConst L{};
    L.w = w;
    L.h = h;
    L.cols = 3 * int64_t(w);
    L.strips = int((L.cols + kLossCols - 1) / kLossCols);
    L.want_grad = grad;
    // Rows per band: a band re-reads 2 r rows, and a launch needs some waves on every SIMD.
    L.band = 32;
    while (L.band > 8 && int64_t(L.strips) * ((h + L.band - 1) / L.band) < kLossFill) L.band /= 2;
    L.lambda = lp->lambda;
    double g[2 * kMaxRadius + 1], sum = 0.0;
    for (int m = -r; m <= r; ++m) {
        g[m + r] = exp(-double(m) * m / (2.0 * double(lp->sigma) * lp->sigma));
        sum += g[m + r];
    }
    for (int m = 0; m <= 2 * r; ++m) L.g[m] = float(g[m] / sum);
    return L;
}

// room for the partial sums: 32 x 8 pixels per set, no more than a workgroup's columns and a shortest band
static int64_t loss_tiles(int32_t w, int32_t h) { return int64_t((w + 31) / 32) * ((h + 7) / 8); }

size_t loss_workspace_bytes(int32_t w, int32_t h)
{
    const size_t maps = align256(size_t(9) * size_t(w) * size_t(h) * 4);
    return maps + align256(size_t(loss_tiles(w, h)) * 6 * 4);
}

template <int R>
static void launch_ssim(const float *img, const float *tgt, float *efg, float *partial, float *grad, int blocks,
                        const LossConst &L, hipStream_t st)
{
    k_ssim_maps<R><<<blocks, 256, 0, st>>>(img, tgt, efg, partial, L);
    if (grad) k_ssim_grad<R><<<blocks, 256, 0, st>>>(img, tgt, efg, grad, L);
}

int launch_loss(const float *img, const float *tgt, int32_t w, int32_t h, const rs_loss_params *lp, float *loss,
                float *grad, void *ws, hipStream_t st)
{
    const LossConst L = loss_const(w, h, lp, grad != nullptr);
    const int64_t blocks = int64_t(L.strips) * ((h + L.band - 1) / L.band);
    float *efg = static_cast<float *>(ws);
    float *partial = reinterpret_cast<float *>(static_cast<char *>(ws) +
                                               align256(size_t(9) * size_t(w) * size_t(h) * 4));
    switch (lp->radius) {
    case 1: launch_ssim<1>(img, tgt, efg, partial, grad, int(blocks), L, st); break;
    case 2: launch_ssim<2>(img, tgt, efg, partial, grad, int(blocks), L, st); break;
    case 3: launch_ssim<3>(img, tgt, efg, partial, grad, int(blocks), L, st); break;
    case 4: launch_ssim<4>(img, tgt, efg, partial, grad, int(blocks), L, st); break;
    case 5: launch_ssim<5>(img, tgt, efg, partial, grad, int(blocks), L, st); break;
    case 6: launch_ssim<6>(img, tgt, efg, partial, grad, int(blocks), L, st); break;
    case 7: launch_ssim<7>(img, tgt, efg, partial, grad, int(blocks), L, st); break;
    default: return RS_ERR_INVALID_ARG;
    }
    k_loss_total<<<1, 256, 0, st>>>(partial, blocks, loss, L);
    return hipGetLastError() == hipSuccess ? RS_OK : RS_ERR_HIP;
}

// ------------------------------------------------ allocation-free variant

// Device scratch of rs_loss_noalloc: a file-scope array each GPU holds for the
// life of the process (its E, F, G maps and per-tile partial sums). Host code
// never passes the array's name to a kernel: it takes the array's device
// address on each device once, with hipGetSymbolAddress, and uses that.
constexpr size_t kLossScratchBytes = size_t(96) << 20;
static __device__ __align__(256) unsigned char scratch[kLossScratchBytes];

constexpr int kMaxScratchDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxScratchDevices];

size_t loss_scratch_bytes() { return kLossScratchBytes; }

// The scratch array's device address on the current device (taken on the first
// call made with that device current).
int loss_scratch(void **out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return RS_ERR_HIP;
    if (dev < 0 || dev >= kMaxScratchDevices) return RS_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return RS_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return RS_OK;
}

}  // namespace rs
