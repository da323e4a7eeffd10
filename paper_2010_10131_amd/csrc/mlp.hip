// Learned cost model of the solver selector (the Sec. IV decision tree's
// role, with an MLP): 10 Table I features -> 32 -> 32 -> 2 (tanh hidden
// layers, linear output = predicted log t_EIG and log t_ALS of one mode).
// Training runs on the device with these kernels:
//   loss/grad  each workgroup takes MS samples through the forward pass, the
//              deltas of L = 0.5/B * sum (Y - T)^2 and the products
//              delta x activation, and writes one partial gradient and loss;
//   reduce     the partial gradients and losses, in workgroup order with
//              FP64 sums (deterministic);
//   Adam       one thread per parameter.
// Parameter packing (float): W1 (32x10, column-major), b1 (32), W2 (32x32),
// b2 (32), W3 (2x32), b3 (2), then the feature normalization mu (10) and
// inverse std (10), which are not trained.
#include "common.h"
#include "internal.h"
#include "selector.h"

namespace sth {

namespace {
constexpr int NI = SEL_IN, NH = SEL_HID, NO = SEL_OUT;
constexpr int OW1 = 0, OB1 = OW1 + NH * NI, OW2 = OB1 + NH, OB2 = OW2 + NH * NH, OW3 = OB2 + NH,
              OB3 = OW3 + NO * NH, OMU = OB3 + NO, OISD = OMU + NI;
constexpr int NTRAIN = OMU;  // trainable parameters
}  // namespace

__global__ void mlp_forward_kernel(const float *__restrict__ w, int64_t B, const float *__restrict__ X,
                                   float *__restrict__ Y) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= B) return;
    float xn[NI], h1[NH], h2[NH];
#pragma unroll
    for (int k = 0; k < NI; ++k) xn[k] = (X[k + NI * s] - w[OMU + k]) * w[OISD + k];
#pragma unroll
    for (int o = 0; o < NH; ++o) {
        float z = w[OB1 + o];
#pragma unroll
        for (int k = 0; k < NI; ++k) z += w[OW1 + o + NH * k] * xn[k];
        h1[o] = tanhf(z);
    }
#pragma unroll
    for (int o = 0; o < NH; ++o) {
        float z = w[OB2 + o];
#pragma unroll
        for (int k = 0; k < NH; ++k) z += w[OW2 + o + NH * k] * h1[k];
        h2[o] = tanhf(z);
    }
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        float z = w[OB3 + o];
#pragma unroll
        for (int k = 0; k < NH; ++k) z += w[OW3 + o + NO * k] * h2[k];
        Y[o + NO * s] = z;
    }
}

// Loss and gradient of MS samples per workgroup.  Bound by latency: a sample
// is 1.4 k multiply-adds, a batch of thousands of samples 40 MFLOP, so the
// work is spread until every workgroup has a few microseconds of it.  A group
// of NH lanes carries one sample, lane o holding neuron o: its rows and
// columns of W2 stay in registers, the sample's activations and deltas cross
// LDS as broadcasts.  Then the 256 threads each own 4 entries of the W2
// gradient (and their share of the rest) and sum delta x activation over the
// MS samples from LDS.  The gradient kept in one thread per parameter, each
// walking all samples serially in 6 workgroups, took nearly all of a
// 1507 us step at 4499 samples; the whole step (this, the reduction, Adam) takes
// 24 us.
// MS = 32: 16 samples doubles the partial gradients to write and read, 64
// leaves half the chip without a workgroup at a few thousand samples.
constexpr int MS = 32, MG = 256 / NH;
// floats of one partial: the trained parameters, then the loss sum (a double)
constexpr int MPART = NTRAIN + 2;
static_assert(NTRAIN % 2 == 0, "the loss sum is 8-byte aligned");

__device__ __forceinline__ float mlp_dot(const float (&w)[NH], const float *__restrict__ v, float z) {
#pragma unroll
    for (int k = 0; k < NH; k += 4) {
        const float4 t = *reinterpret_cast<const float4 *>(v + k);
        z += w[k] * t.x;
        z += w[k + 1] * t.y;
        z += w[k + 2] * t.z;
        z += w[k + 3] * t.w;
    }
    return z;
}

// One workgroup per MS samples.  part: MPART floats per workgroup, or null
// (a single workgroup): the sums go to grad and loss directly.
__global__ __launch_bounds__(256) void mlp_grad_kernel(const float *__restrict__ w, int64_t B,
                                                       const float *__restrict__ X, const float *__restrict__ T,
                                                       float *__restrict__ part, float *__restrict__ grad,
                                                       float *__restrict__ loss) {
    __shared__ __align__(16) float s_x[MS][12], s_h1[MS][NH], s_h2[MS][NH], s_d1[MS][NH], s_d2[MS][NH], s_d3[MS][NO];
    __shared__ double s_l[MS];
    const int tid = threadIdx.x, o = tid % NH, grp = tid / NH;
    const int64_t s0 = (int64_t)blockIdx.x * MS;
    const int ns = (int)(B - s0 < MS ? B - s0 : MS);
    float w1[NI], wr[NH], wc[NH];
#pragma unroll
    for (int k = 0; k < NI; ++k) w1[k] = w[OW1 + o + NH * k];
#pragma unroll
    for (int k = 0; k < NH; ++k) {
        wr[k] = w[OW2 + o + NH * k];   // row o (forward)
        wc[k] = w[OW2 + k + NH * o];   // column o (backward)
    }
    const float b1 = w[OB1 + o], b2 = w[OB2 + o];
    const float w30 = w[OW3 + NO * o], w31 = w[OW3 + 1 + NO * o];
    for (int e = tid; e < MS * NI; e += 256) {
        const int sl = e / NI, k = e - sl * NI;
        s_x[sl][k] = sl < ns ? (X[k + NI * (s0 + sl)] - w[OMU + k]) * w[OISD + k] : 0.f;
    }
    __syncthreads();
    // the groups are halves of a wave: a wave's own LDS writes are visible to
    // it in order, so only the compiler needs the fences between the layers
    for (int sl = grp; sl < MS; sl += MG) {
        float z = b1;
#pragma unroll
        for (int k = 0; k < NI; ++k) z += w1[k] * s_x[sl][k];
        const float h1 = sl < ns ? tanhf(z) : 0.f;   // samples past the batch contribute nothing
        s_h1[sl][o] = h1;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const float h2 = sl < ns ? tanhf(mlp_dot(wr, s_h1[sl], b2)) : 0.f;
        s_h2[sl][o] = h2;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (o < NO) {
            float y = w[OB3 + o];
            for (int k = 0; k < NH; ++k) y += w[OW3 + o + NO * k] * s_h2[sl][k];
            const float r = sl < ns ? y - T[o + NO * (s0 + (sl < ns ? sl : 0))] : 0.f;
            s_d3[sl][o] = r * (1.0f / (float)B);
            const double r2 = (double)r * (double)r;
            const double both = r2 + __shfl_xor(r2, 1);
            if (o == 0) s_l[sl] = both;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const float d2 = sl < ns ? (w30 * s_d3[sl][0] + w31 * s_d3[sl][1]) * (1.0f - h2 * h2) : 0.f;
        s_d2[sl][o] = d2;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        s_d1[sl][o] = sl < ns ? mlp_dot(wc, s_d2[sl], 0.f) * (1.0f - h1 * h1) : 0.f;
    }
    __syncthreads();
    float *const out = part ? part + (int64_t)blockIdx.x * MPART : grad;
    // W2: rows o, columns 4 grp .. 4 grp + 3 (samples past ns have zero deltas)
    static_assert(MG * 4 == NH, "four columns per group");
    float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int sl = 0; sl < MS; ++sl) {
        const float d = s_d2[sl][o];
        const float4 h = *reinterpret_cast<const float4 *>(&s_h1[sl][4 * grp]);
        a[0] += d * h.x;
        a[1] += d * h.y;
        a[2] += d * h.z;
        a[3] += d * h.w;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) out[OW2 + o + NH * (4 * grp + c)] = a[c];
    // W1 (rows o, columns grp, grp + MG), the biases and W3
    for (int k = grp; k < NI; k += MG) {
        float g = 0.f;
#pragma unroll 8
        for (int sl = 0; sl < MS; ++sl) g += s_d1[sl][o] * s_x[sl][k];
        out[OW1 + o + NH * k] = g;
    }
    float g = 0.f;
    if (grp == 2) {
        for (int sl = 0; sl < MS; ++sl) g += s_d1[sl][o];
        out[OB1 + o] = g;
    } else if (grp == 3) {
        for (int sl = 0; sl < MS; ++sl) g += s_d2[sl][o];
        out[OB2 + o] = g;
    } else if (grp == 4 || grp == 5) {
        for (int sl = 0; sl < MS; ++sl) g += s_d3[sl][grp - 4] * s_h2[sl][o];
        out[OW3 + (grp - 4) + NO * o] = g;
    } else if (grp == 6 && o < NO) {
        for (int sl = 0; sl < MS; ++sl) g += s_d3[sl][o];
        out[OB3 + o] = g;
    } else if (grp == 7 && o == 0) {
        double l = 0.0;
        for (int sl = 0; sl < ns; ++sl) l += s_l[sl];
        if (part) *reinterpret_cast<double *>(out + NTRAIN) = l;
        else if (loss) *loss = (float)(0.5 * l / (double)B);
    }
    if (!part)
        for (int p = NTRAIN + tid; p < SEL_NPARAM; p += 256) grad[p] = 0.f;
}

// grad = the partial gradients summed over the np workgroups (64 parameters
// per workgroup, four waves on interleaved partials, FP64 sums combined in a
// fixed order), the normalization entries zero; loss from the partial sums.
__global__ __launch_bounds__(256) void mlp_reduce_kernel(const float *__restrict__ part, int np, int64_t B,
                                                         float *__restrict__ grad, float *__restrict__ loss) {
    __shared__ double s_sum[4][64];
    const int el = threadIdx.x & 63, ks = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + el;
    const bool is_loss = p == SEL_NPARAM;   // one past the parameters: the loss
    double acc = 0.0;
    if (p < NTRAIN) {
#pragma unroll 8
        for (int k = ks; k < np; k += 4) acc += (double)part[(int64_t)k * MPART + p];
    } else if (is_loss) {
        for (int k = ks; k < np; k += 4) acc += *reinterpret_cast<const double *>(part + (int64_t)k * MPART + NTRAIN);
    }
    s_sum[ks][el] = acc;
    __syncthreads();
    if (ks != 0) return;
    const double sum = (s_sum[0][el] + s_sum[1][el]) + (s_sum[2][el] + s_sum[3][el]);
    if (p < SEL_NPARAM) grad[p] = p < NTRAIN ? (float)sum : 0.f;
    else if (is_loss && loss) *loss = (float)(0.5 * sum / (double)B);
}

__global__ void adam_kernel(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m,
                            float *__restrict__ v, int64_t n, float lr, float b1, float b2, float eps,
                            float c1, float c2) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const float gp = g[p];
    const float mp = b1 * m[p] + (1.0f - b1) * gp;
    const float vp = b2 * v[p] + (1.0f - b2) * gp * gp;
    m[p] = mp;
    v[p] = vp;
    w[p] -= lr * (mp * c1) / (sqrtf(vp * c2) + eps);
}

// workspace floats per sample: more than the partial gradients take
constexpr int64_t MLP_WS_FLOATS = NI + 2 * NH + NO + 2 * NH + NO;
size_t mlp_ws_bytes(int64_t B) {
    return (size_t)B * MLP_WS_FLOATS * sizeof(float) + 256;
}

hipError_t mlp_forward_launch(const float *w, int64_t B, const float *X, float *Y, void *ws, hipStream_t s) {
    const unsigned g = (unsigned)((B + 255) / 256);
    hipLaunchKernelGGL(mlp_forward_kernel, dim3(g), dim3(256), 0, s, w, B, X, Y);
    return hipGetLastError();
}

hipError_t mlp_loss_grad_launch(const float *w, int64_t B, const float *X, const float *T, float *grad,
                                float *loss, void *ws, hipStream_t s) {
    const int64_t np = (B + MS - 1) / MS;
    float *part = np > 1 ? (float *)ws : nullptr;   // np MPART floats, below mlp_ws_bytes(B) for B > MS
    static_assert((int64_t)2 * MPART <= (int64_t)(MS + 1) * MLP_WS_FLOATS && MPART <= MS * MLP_WS_FLOATS,
                  "the partial gradients fit the workspace");
    hipLaunchKernelGGL(mlp_grad_kernel, dim3((unsigned)np), dim3(256), 0, s, w, B, X, T, part, grad, loss);
    if (np > 1)
        hipLaunchKernelGGL(mlp_reduce_kernel, dim3((SEL_NPARAM + 64) / 64), dim3(256), 0, s, part, (int)np, B, grad,
                           loss);
    return hipGetLastError();
}

hipError_t adam_launch(float *w, const float *g, float *m, float *v, int64_t n, float lr, float b1,
                       float b2, float eps, int step, hipStream_t s) {
    const float c1 = 1.0f / (1.0f - powf(b1, (float)step));
    const float c2 = 1.0f / (1.0f - powf(b2, (float)step));
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w, g, m, v, n, lr,
                       b1, b2, eps, c1, c2);
    return hipGetLastError();
}

int mlp_num_trainable() { return NTRAIN; }

}  // namespace sth
