// lbm_mlp.hip -- learned eddy-viscosity closure: parameter packing, the
// standalone inference kernel (same device code as the fused collision), the
// training samples of a filtered fine lattice (its filter is k_filter in
// lbm_kernels.h), and the FP32 training kernels (forward, backward,
// deterministic gradient reduction, Adam).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "lbm.h"
#include "lbm_internal.h"
#include "lbm_mlp_device.h"

using namespace lbmd;

lbm_status lbmd_fail_hip(lbm_lattice *lat, hipError_t e, const char *what);
lbm_status lbmd_set_err(lbm_status s, const char *msg);
lbm_config lbmd_config(const lbm_lattice *lat);
hipStream_t lbmd_stream(const lbm_lattice *lat);
bool lbmd_failed(const lbm_lattice *lat);
void lbmd_set_mlp(lbm_lattice *lat, void *block, const MlpDev &m);
void *lbmd_mlp_block(lbm_lattice *lat);
void lbmd_clear_mlp(lbm_lattice *lat);
lbm_status lbmd_filter(lbm_lattice *lat, int factor, lbm_status (*targets)(lbm_lattice *, const double *, int, void *),
                       void *arg);

#define HIPCHK(lat, expr)                                              \
    do {                                                               \
        hipError_t e_ = (expr);                                        \
        if (e_ != hipSuccess) return lbmd_fail_hip((lat), e_, #expr);  \
    } while (0)

namespace {

// Offsets in the packed FP32 parameter vector (see lbm.h).
constexpr int OW1 = 0, OB1 = 224, OW2 = 256, OB2 = 1280, OW3 = 1312, OB3 = 1344, OMEAN = 1345, OSTD = 1352;
constexpr int NP = LBM_MLP_NPARAMS;   // 1359
constexpr int NTRAIN = 1345;          // trainable entries (weights and biases)

// FP32 -> BF16 bit pattern, round to nearest even (NaN kept quiet).
uint16_t bf16_bits(float v) {
    uint32_t b;
    std::memcpy(&b, &v, 4);
    if ((b & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((b >> 16) | 0x40u);
    b += 0x7fffu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}

// Device block (see MlpDev): w1p[32][8] u16 | w2p[2][2][32][8] u16 | w3p[2][16] u16 |
// b1p[2][16] b2p[2][16] b3[1] pad[3] mean[7] pad inv_sd[7] pad (floats).  "Accumulator
// order" of lane group g: entry r is neuron 8 (r / 4) + 4 g + r % 4 (lbm_mlp_device.h).
constexpr size_t kW3Off = (256 + 1024) * 2, kFloatOff = kW3Off + 32 * 2;
constexpr size_t kBlockBytes = kFloatOff + (32 + 32 + 4 + 8 + 8) * 4;

int acc_neuron(int r, int g) { return 8 * (r / 4) + 4 * g + (r % 4); }

void pack_block(const float *P, std::vector<unsigned char> &out) {
    out.assign(kBlockBytes, 0);
    uint16_t *w1p = reinterpret_cast<uint16_t *>(out.data());
    uint16_t *w2p = w1p + 256;
    uint16_t *w3p = reinterpret_cast<uint16_t *>(out.data() + kW3Off);
    float *fl = reinterpret_cast<float *>(out.data() + kFloatOff);
    for (int o = 0; o < 32; ++o)
        for (int s = 0; s < 8; ++s) w1p[o * 8 + s] = s < 7 ? bf16_bits(P[OW1 + o * 7 + s]) : 0;
    // W2 as the A operands of the two layer-2 products: product p, lane group g,
    // row i, K slot s holds W2[i][neuron], the neuron that accumulator register
    // 8p + s of lane group g holds after layer 1
    for (int pr = 0; pr < 2; ++pr)
        for (int g = 0; g < 2; ++g)
            for (int i = 0; i < 32; ++i)
                for (int s = 0; s < 8; ++s)
                    w2p[((pr * 2 + g) * 32 + i) * 8 + s] = bf16_bits(P[OW2 + i * 32 + acc_neuron(8 * pr + s, g)]);
    for (int g = 0; g < 2; ++g)
        for (int r = 0; r < 16; ++r) {
            const int o = acc_neuron(r, g);
            w3p[g * 16 + r] = bf16_bits(P[OW3 + o]);
            fl[g * 16 + r] = P[OB1 + o];
            fl[32 + g * 16 + r] = P[OB2 + o];
        }
    fl[64] = P[OB3];
    for (int k = 0; k < 7; ++k) {
        fl[68 + k] = P[OMEAN + k];
        fl[76 + k] = 1.0f / P[OSTD + k];
    }
}

MlpDev block_view(void *d) {
    MlpDev m;
    unsigned char *b = static_cast<unsigned char *>(d);
    float *fl = reinterpret_cast<float *>(b + kFloatOff);
    m.w1 = reinterpret_cast<uint16_t *>(b);
    m.w2 = m.w1 + 256;
    m.w3 = reinterpret_cast<uint16_t *>(b + kW3Off);
    m.b1 = fl;
    m.b2 = fl + 32;
    m.b3 = fl + 64;
    m.mean = fl + 68;
    m.inv_sd = fl + 76;
    return m;
}

lbm_status check_params(const float *P) {
    for (int k = 0; k < NP; ++k)
        if (!std::isfinite(P[k])) return lbmd_set_err(LBM_EINVAL, "closure parameters must be finite");
    for (int k = 0; k < 7; ++k)
        if (!(P[OSTD + k] > 0.0f)) return lbmd_set_err(LBM_EINVAL, "closure std entries must be > 0");
    return LBM_OK;
}

}  // namespace

void lbmd_free_mlp(lbm_lattice *lat) {
    void *b = lbmd_mlp_block(lat);
    if (b) (void)hipFree(b);
    lbmd_clear_mlp(lat);
}

extern "C" lbm_status lbm_set_mlp(lbm_lattice *lat, const float *params_host, size_t n) {
    if (!lat) return lbmd_set_err(LBM_EINVAL, "null lattice handle");
    if (lbmd_failed(lat)) return lbmd_set_err(LBM_ESTATE, "lattice handle failed earlier");
    if (!params_host || n != (size_t)NP) return lbmd_set_err(LBM_EINVAL, "expected LBM_MLP_NPARAMS floats");
    lbm_status s = check_params(params_host);
    if (s != LBM_OK) return s;
    std::vector<unsigned char> blk;
    pack_block(params_host, blk);
    void *d = lbmd_mlp_block(lat);
    if (!d) HIPCHK(lat, hipMalloc(&d, kBlockBytes));
    hipStream_t st = lbmd_stream(lat);
    hipError_t e = hipMemcpyAsync(d, blk.data(), kBlockBytes, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        (void)hipFree(d);
        lbmd_clear_mlp(lat);
        return lbmd_fail_hip(lat, e, "closure upload");
    }
    lbmd_set_mlp(lat, d, block_view(d));
    return LBM_OK;
}

// ------------------------------------------------------------ inference
namespace lbmd {
__global__ __launch_bounds__(256) void k_mlp_infer(MlpDev m, float nu0, const float *feat, long long n,
                                                   float *nut) {
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    float x[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) x[k] = t < n ? feat[t * 7 + k] : m.mean[k];
    const float sp = mlp_wave_eval(m, x);  // every lane takes part
    if (t < n) nut[t] = nu0 * sp;
}
}  // namespace lbmd

extern "C" lbm_status lbm_mlp_infer(const float *params_host, double nu0, const float *feat_dev, int64_t n,
                                    float *nut_dev, void *hip_stream) {
    if (!params_host || (n > 0 && (!feat_dev || !nut_dev)) || n < 0)
        return lbmd_set_err(LBM_EINVAL, "bad arguments to lbm_mlp_infer");
    lbm_status s = check_params(params_host);
    if (s != LBM_OK) return s;
    if (n == 0) return LBM_OK;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    std::vector<unsigned char> blk;
    pack_block(params_host, blk);
    void *d = nullptr;
    HIPCHK(nullptr, hipMalloc(&d, kBlockBytes));
    hipError_t e = hipMemcpyAsync(d, blk.data(), kBlockBytes, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) {
        k_mlp_infer<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(block_view(d), (float)nu0, feat_dev, n, nut_dev);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    (void)hipFree(d);
    if (e != hipSuccess) return lbmd_fail_hip(nullptr, e, "lbm_mlp_infer");
    return LBM_OK;
}

// ------------------------------------------------------------ box filter
namespace lbmd {
// coarse: FP64 planes rho_bar, U (3), T (6: xx yy zz xy xz yz) per coarse node (k_filter).
__global__ __launch_bounds__(256) void k_closure_targets(const double *coarse, int cx, int cy, int cz, double nu_c,
                                                         float *feat, float *target) {
    const long long nc = (long long)cx * cy * cz;
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= nc) return;
    const int X = (int)(t % cx), Y = (int)((t / cx) % cy), Z = (int)(t / ((long long)cx * cy));
    auto at = [&](int comp, int x, int y, int z) {
        x = (x + cx) % cx;
        y = (y + cy) % cy;
        z = (z + cz) % cz;
        return coarse[comp * nc + ((long long)z * cy + y) * cx + x];
    };
    // G[a][b] = dU_b / dx_a, second-order central differences.
    double G[3][3];
    for (int b = 0; b < 3; ++b) {
        G[0][b] = 0.5 * (at(1 + b, X + 1, Y, Z) - at(1 + b, X - 1, Y, Z));
        G[1][b] = 0.5 * (at(1 + b, X, Y + 1, Z) - at(1 + b, X, Y - 1, Z));
        G[2][b] = 0.5 * (at(1 + b, X, Y, Z + 1) - at(1 + b, X, Y, Z - 1));
    }
    double S[3][3];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) S[a][b] = 0.5 * (G[a][b] + G[b][a]);
    const double T[3][3] = {{coarse[4 * nc + t], coarse[7 * nc + t], coarse[8 * nc + t]},
                            {coarse[7 * nc + t], coarse[5 * nc + t], coarse[9 * nc + t]},
                            {coarse[8 * nc + t], coarse[9 * nc + t], coarse[6 * nc + t]}};
    const double tr = (T[0][0] + T[1][1] + T[2][2]) / 3.0;
    double num = 0.0, ss = 0.0;
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) {
            num += (T[a][b] - (a == b ? tr : 0.0)) * S[a][b];
            ss += S[a][b] * S[a][b];
        }
    const double nut = fmax(0.0, -num / (2.0 * ss + 1e-30));
    const double rho = coarse[t];
    const double tau_e = 3.0 * (nu_c + nut) + 0.5;
    const double c = -(2.0 / 3.0) * rho * tau_e;
    feat[t * 7 + 0] = (float)(c * S[0][0]);
    feat[t * 7 + 1] = (float)(c * S[1][1]);
    feat[t * 7 + 2] = (float)(c * S[2][2]);
    feat[t * 7 + 3] = (float)(c * S[0][1]);
    feat[t * 7 + 4] = (float)(c * S[0][2]);
    feat[t * 7 + 5] = (float)(c * S[1][2]);
    feat[t * 7 + 6] = (float)rho;
    target[t] = (float)(nut / nu_c);
}
}  // namespace lbmd

extern "C" lbm_status lbm_filter_snapshot(lbm_lattice *fine, int factor, float *feat_dev, float *target_dev) {
    if (!fine) return lbmd_set_err(LBM_EINVAL, "null lattice handle");
    if (lbmd_failed(fine)) return lbmd_set_err(LBM_ESTATE, "lattice handle failed earlier");
    const lbm_config c = lbmd_config(fine);
    if (factor < 1 || c.nx % factor || c.ny % factor || c.nz % factor)
        return lbmd_set_err(LBM_EINVAL, "lattice sizes must be divisible by the filter factor");
    if (!feat_dev || !target_dev) return lbmd_set_err(LBM_EINVAL, "null output");
    struct Out {
        float *feat, *target;
    } out{feat_dev, target_dev};
    return lbmd_filter(
        fine, factor,
        [](lbm_lattice *lat, const double *coarse, int f, void *arg) -> lbm_status {
            const lbm_config c = lbmd_config(lat);
            const Out *o = static_cast<const Out *>(arg);
            const int cx = c.nx / f, cy = c.ny / f, cz = c.nz / f;
            const double nu_c = (c.tau - 0.5) / 3.0 / f;
            const unsigned blocks = (unsigned)(((long long)cx * cy * cz + 255) / 256);
            k_closure_targets<<<blocks, 256, 0, lbmd_stream(lat)>>>(coarse, cx, cy, cz, nu_c, o->feat, o->target);
            HIPCHK(lat, hipGetLastError());
            return LBM_OK;
        },
        &out);
}

// ------------------------------------------------------------ training
namespace lbmd {
constexpr int kTrainSamples = 128;  // samples a block works on at a time, 32 a wave
constexpr int kTrainPitch = 33;     // LDS row of one sample (32 neurons and a pad: no bank conflicts)

// Forward and backward of 128 samples per block and pass on FP32 matrix cores
// (v_mfma_f32_32x32x2f32: FP32 operands, products and sums), and the block's sum
// of the gradient in part[block][NP + 1] (packed parameter order, then the loss).
// Bound by latency: the 4096 samples of a mini-batch are 31 MFLOP, 32 blocks; one
// thread per sample with its record in memory and one thread per parameter and 256
// samples took 21 + 123 us a batch, this 13 (with the parameters staged through
// LDS first, and the next indices loaded ahead, 13.7).
//
// Layouts: neurons are the M dimension, samples the N dimension, so accumulator
// register r of lane l holds neuron nr(r) = 8 (r / 4) + 4 (l / 32) + r % 4 of
// sample l % 32.  The next product takes register r as its B operand as it is
// (lane half g the K slot of neuron nr(r)), with the weights' columns in the same
// order.  The gradient products sum over samples, so their operands go through
// LDS: wave 0 forms dW2 = d2 h1^T, waves 1, 2 and 3 the products of d1, d2 and h2
// with X = [x, 1, d3] (dW1 and db1, db2, dW3).
__global__ __launch_bounds__(256) void k_train(const float *P, const float *feat, const float *target,
                                               const long long *idx, long long base, int nb, long long n, float scale,
                                               float *part) {
    __shared__ float sh[4][kTrainSamples * kTrainPitch];  // d2, d1, h2, h1
    __shared__ float sx[kTrainSamples * 9];
    __shared__ float s_sum[4][2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 5, c = lane & 31;
    auto nr = [&](int r) { return 8 * (r / 4) + 4 * g + (r % 4); };

    float w1[4], w2[16], w2t[16], w3[16], mean[4], sd[4];
    f32x16 b1, b2;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = 2 * j + g;
        w1[j] = k < 7 ? P[OW1 + c * 7 + k] : 0.0f;
        mean[j] = k < 7 ? P[OMEAN + k] : 0.0f;
        sd[j] = k < 7 ? P[OSTD + k] : 1.0f;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        w2[r] = P[OW2 + c * 32 + nr(r)];
        w2t[r] = P[OW2 + nr(r) * 32 + c];
        w3[r] = P[OW3 + nr(r)];
        b1[r] = P[OB1 + nr(r)];
        b2[r] = P[OB2 + nr(r)];
    }
    const float b3 = P[OB3];
    const f32x16 zero = {};
    f32x16 acc = zero;
    float lsum = 0.0f, dsum = 0.0f;
    for (int b0 = blockIdx.x * kTrainSamples; b0 < nb; b0 += gridDim.x * kTrainSamples) {
        const int sl = wave * 32 + c;  // the lane's sample in the block
        const int b = b0 + sl;
        long long s = b < nb ? (idx ? idx[base + b] : base + b) : -1;
        const bool use = s >= 0 && s < n;  // an out-of-range sample contributes nothing
        if (!use) s = 0;
        float x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 2 * j + g;
            x[j] = use && k < 7 ? (feat[s * 7 + k] - mean[j]) / sd[j] : 0.0f;
        }
        const float t = use ? target[s] : 0.0f;
        f32x16 z1 = b1, z2 = b2, d1 = zero;
#pragma unroll
        for (int j = 0; j < 4; ++j) z1 = __builtin_amdgcn_mfma_f32_32x32x2f32(w1[j], x[j], z1, 0, 0, 0);
        float h1[16], h2[16], d2[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) h1[r] = z1[r] > 0.0f ? z1[r] : 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) z2 = __builtin_amdgcn_mfma_f32_32x32x2f32(w2[r], h1[r], z2, 0, 0, 0);
        float z3 = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            h2[r] = z2[r] > 0.0f ? z2[r] : 0.0f;
            z3 += w3[r] * h2[r];
        }
        z3 += __shfl_xor(z3, 32, 64);
        z3 += b3;
        const float res = softplus_f(z3) - t;
        const float sig = 1.0f / (1.0f + expf(-z3));
        const float d3 = use ? scale * 2.0f * res * sig : 0.0f;
        if (g == 0) {
            lsum += use ? scale * res * res : 0.0f;
            dsum += d3;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            d2[r] = z2[r] > 0.0f ? d3 * w3[r] : 0.0f;
            d1 = __builtin_amdgcn_mfma_f32_32x32x2f32(w2t[r], d2[r], d1, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int a = sl * kTrainPitch + nr(r);
            sh[0][a] = d2[r];
            sh[1][a] = z1[r] > 0.0f ? d1[r] : 0.0f;
            sh[2][a] = h2[r];
            sh[3][a] = h1[r];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) sx[sl * 9 + 2 * j + g] = 2 * j + g < 7 ? x[j] : 1.0f;
        if (g == 0) sx[sl * 9 + 8] = d3;
        __syncthreads();
        const float *sa = sh[wave == 0 || wave == 2 ? 0 : (wave == 1 ? 1 : 2)];
#pragma unroll 8
        for (int j = 0; j < kTrainSamples / 2; ++j) {
            const int q = 2 * j + g;
            const float bv = wave == 0 ? sh[3][q * kTrainPitch + c] : (c < 9 ? sx[q * 9 + c] : 0.0f);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(sa[q * kTrainPitch + c], bv, acc, 0, 0, 0);
        }
        __syncthreads();
    }
    // acc[r]: row nr(r) (neuron), column c
    float *out = part + (long long)blockIdx.x * (NP + 1);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int o = nr(r);
        if (wave == 0) out[OW2 + o * 32 + c] = acc[r];
        else if (wave == 1 && c < 8) out[c < 7 ? OW1 + o * 7 + c : OB1 + o] = acc[r];
        else if (wave == 2 && c == 7) out[OB2 + o] = acc[r];
        else if (wave == 3 && c == 8) out[OW3 + o] = acc[r];
    }
    for (int o = 32; o > 0; o >>= 1) {
        lsum += __shfl_xor(lsum, o, 64);
        dsum += __shfl_xor(dsum, o, 64);
    }
    if (lane == 0) s_sum[wave][0] = lsum, s_sum[wave][1] = dsum;
    __syncthreads();
    if (threadIdx.x < 14) out[OMEAN + threadIdx.x] = 0.0f;  // mean and std are not trained
    if (threadIdx.x == 0) {
        out[NP] = (s_sum[0][0] + s_sum[1][0]) + (s_sum[2][0] + s_sum[3][0]);
        out[OB3] = (s_sum[0][1] + s_sum[1][1]) + (s_sum[2][1] + s_sum[3][1]);
    }
}

// Plain zero fill (used instead of memset so callers may capture the work).
__global__ __launch_bounds__(256) void k_zero(float *p, long long n) {
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t < n) p[t] = 0.0f;
}

// Sum of the block partials of parameter k = 64 blockIdx.x + thread % 64: four
// runs of rows, each in order, then the runs in order.  Valid in threads 0..63.
__device__ __forceinline__ float row_sum(const float *part, int rows, int k) {
    __shared__ float s[4][64];
    const int run = threadIdx.x >> 6, per = (rows + 3) / 4;
    const int r0 = run * per, r1 = min(rows, r0 + per);
    float g = 0.0f;
    if (k <= NP) {
#pragma unroll 8
        for (int c = r0; c < r1; ++c) g += part[(long long)c * (NP + 1) + k];
    }
    s[run][threadIdx.x & 63] = g;
    __syncthreads();
    const int t = threadIdx.x & 63;
    return (s[0][t] + s[1][t]) + (s[2][t] + s[3][t]);
}

// Gradient and loss from the block partials.
__global__ __launch_bounds__(256) void k_grad_sum(const float *part, int rows, float *grad, float *loss) {
    const int k = blockIdx.x * 64 + (threadIdx.x & 63);
    const float g = row_sum(part, rows, k);
    if (threadIdx.x >= 64 || k > NP) return;
    if (k == NP) *loss = g;
    else grad[k] = g;
}

// One Adam step from the block partials; loss_log[epoch] += batch loss * w.
__global__ __launch_bounds__(256) void k_adam(const float *part, int rows, float *P, float *m, float *v, float lr,
                                              float bc1, float bc2, float *loss_log, int epoch, float w) {
    const int k = blockIdx.x * 64 + (threadIdx.x & 63);
    const float g = row_sum(part, rows, k);
    if (threadIdx.x >= 64 || k > NP) return;
    if (k == NP) {
        loss_log[epoch] += g * w;
        return;
    }
    if (k >= NTRAIN) return;
    const float mk = 0.9f * m[k] + 0.1f * g;
    const float vk = 0.999f * v[k] + 0.001f * g * g;
    m[k] = mk;
    v[k] = vk;
    P[k] -= lr * (mk / bc1) / (sqrtf(vk / bc2) + 1e-8f);
}
constexpr int kParamBlocks = (NP + 1 + 63) / 64;
}  // namespace lbmd

namespace {
struct TrainScratch {
    float *p = nullptr;
    ~TrainScratch() {
        if (p) (void)hipFree(p);
    }
};

// Blocks of k_train: one per 128 samples up to 256, beyond that one per 8192.  A gradient
// entry is an FP32 sum over all samples of its block (one wave's accumulator), then
// over the blocks in four runs.
int train_blocks(long long n) {
    const long long b = (n + kTrainSamples - 1) / kTrainSamples;
    return (int)std::min(b, std::max(256ll, n / 8192));
}
}  // namespace

extern "C" lbm_status lbm_mlp_grad(const float *params_dev, const float *feat_dev, const float *target_dev, int64_t n,
                                   float *grad_dev, float *loss_dev, void *hip_stream) {
    if (!params_dev || !feat_dev || !target_dev || !grad_dev || !loss_dev || n < 1)
        return lbmd_set_err(LBM_EINVAL, "bad arguments to lbm_mlp_grad");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    // sub-ranges of 2^30 samples (32-bit counts in the kernel), each with its own rows
    constexpr long long SUB = 1ll << 30;
    int rows = 0;
    for (long long b = 0; b < n; b += SUB) rows += train_blocks(std::min<long long>(SUB, n - b));
    TrainScratch sc;
    HIPCHK(nullptr, hipMalloc(&sc.p, (size_t)rows * (NP + 1) * sizeof(float)));
    int row = 0;
    for (long long b = 0; b < n; b += SUB) {
        const int nb = (int)std::min<long long>(SUB, n - b), blocks = train_blocks(nb);
        k_train<<<blocks, 256, 0, st>>>(params_dev, feat_dev, target_dev, nullptr, b, nb, n, 1.0f / (float)n,
                                        sc.p + (long long)row * (NP + 1));
        row += blocks;
    }
    k_grad_sum<<<kParamBlocks, 256, 0, st>>>(sc.p, rows, grad_dev, loss_dev);
    HIPCHK(nullptr, hipGetLastError());
    HIPCHK(nullptr, hipStreamSynchronize(st));
    return LBM_OK;
}

extern "C" lbm_status lbm_mlp_train(float *params_dev, const float *feat_dev, const float *target_dev, int64_t n,
                                    const int64_t *perm_dev, int batch, int epochs, double lr, float *loss_log_dev,
                                    void *hip_stream) {
    if (!params_dev || !feat_dev || !target_dev || !perm_dev || !loss_log_dev || n < 1 || batch < 1 ||
        batch > 65536 || epochs < 0 || !(lr > 0.0))
        return lbmd_set_err(LBM_EINVAL, "bad arguments to lbm_mlp_train");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    // Adam's two moments, then the block partials
    TrainScratch sc;
    HIPCHK(nullptr, hipMalloc(&sc.p, (size_t)(2 * NP + train_blocks(batch) * (NP + 1)) * sizeof(float)));
    float *m = sc.p, *v = m + NP, *part = v + NP;
    k_zero<<<(2 * NP + 255) / 256, 256, 0, st>>>(m, 2 * NP);
    k_zero<<<(unsigned)((epochs + 255) / 256 + 1), 256, 0, st>>>(loss_log_dev, epochs);
    const long long nbatches = (n + batch - 1) / batch;
    long long step = 0;
    for (int ep = 0; ep < epochs; ++ep) {
        for (long long bi = 0; bi < nbatches; ++bi) {
            const long long base = bi * batch;
            const int nb = (int)std::min<long long>(batch, n - base), rows = train_blocks(nb);
            k_train<<<rows, 256, 0, st>>>(params_dev, feat_dev, target_dev,
                                          reinterpret_cast<const long long *>(perm_dev), (long long)ep * n + base, nb,
                                          n, 1.0f / nb, part);
            ++step;
            const float bc1 = 1.0f - std::pow(0.9f, (float)step);
            const float bc2 = 1.0f - std::pow(0.999f, (float)step);
            k_adam<<<kParamBlocks, 256, 0, st>>>(part, rows, params_dev, m, v, (float)lr, bc1, bc2, loss_log_dev, ep,
                                                 1.0f / (float)nbatches);
        }
        HIPCHK(nullptr, hipGetLastError());
    }
    HIPCHK(nullptr, hipStreamSynchronize(st));
    return LBM_OK;
}
