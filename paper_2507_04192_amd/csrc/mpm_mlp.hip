// Learned field alpha(x) ~ N_theta(x) (Sec. 3.2, eq:nn_apprx): a small MLP
// whose layers run on the matrix cores of gfx950.
//
// A layer h' = act(h W^T + b) is a product computed as 16 x 16 output tiles
// with gfx950's v_mfma_f32_16x16x32_bf16 (BF16 operands, FP32 accumulation,
// 32-deep K steps) or v_mfma_f32_16x16x4_f32 (FP32 operands).  Weights and
// activations are staged in LDS, zero-padded to the step (16 or 32), by
// workgroups of 64 samples.  The backward pass is one kernel: a workgroup
// carries its samples' layer adjoints dZ down the layers in LDS and forms the
// weight gradients dW = dZ^T H (a reduction over samples) of its samples on
// the way; a second kernel sums the workgroups' gradients in a fixed order.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>

#include "../../include/mpm.h"

namespace mpm {
void set_global_error(const char* msg);
}

// Work buffer of mpm_mlp_backward_noalloc (the workgroups' gradients), a
// file-scope device array: every GPU the library runs on holds one copy
// for the life of the process.  Host code never passes this name to a
// kernel (on the host it is a stand-in, not a device address); it uses the
// per-device address from hipGetSymbolAddress below.
static __device__ __align__(256) float scratch[MPM_MLP_SCRATCH_FLOATS];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_ptr[kMaxDevices] = {};

// Device address of this device's scratch array, looked up once per device
// (with that device current) and kept.
int scratch_address(float** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        mpm::set_global_error("mpm_mlp_backward_noalloc: no usable current device");
        return MPM_EHIP;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            mpm::set_global_error("mpm_mlp_backward_noalloc: hipGetSymbolAddress of the scratch array failed");
            return MPM_EHIP;
        }
        g_scratch_ptr[dev] = (float*)p;
    }
    *out = g_scratch_ptr[dev];
    return MPM_OK;
}

constexpr int kMaxW = 128;
constexpr int kRows = 64;        // samples of a workgroup
constexpr int kPad = 32;         // operands are zero-padded to this many columns
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));

struct MlpDesc {
    int L;
    int w[MPM_MLP_MAX_LAYERS + 1];    // true widths
    int offW[MPM_MLP_MAX_LAYERS], offb[MPM_MLP_MAX_LAYERS];
    long long offC[MPM_MLP_MAX_LAYERS];   // per-layer offset in the cache (per sample count n)
    int out_act;
    int hidden_act;                   // MPM_HIDDEN_TANH or MPM_HIDDEN_RELU
    float scale, shift;
    float in_scale[MPM_MLP_MAX_IN], in_shift[MPM_MLP_MAX_IN];
};

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Operands of a 16 x 16 tile C[r][c] = sum_k A(r, k) B(k, c).  Lane l holds
// C[4*(l/16) + i][l%16], i = 0..3.  FP32: lane l supplies A(l%16, k) and
// B(k, l%16) for k = k0 + l/16 of each 4-deep step.  BF16: the eight
// k = k0 + 8*(l/16) + i of each 32-deep step, rounded to nearest even (the
// same k for both operands, so the pairing is exact whatever order the unit
// sums in).
template <int BF16> struct Opnd;
template <> struct Opnd<0> {
    static constexpr int STEP = 4, GROUP = 8;   // steps issued together
    typedef float V;
    // element k of the lane's vector at p (k advances by `stride` elements)
    static __device__ __forceinline__ V load(const float* p, int) { return *p; }
    static __device__ __forceinline__ f4 mma(V a, V b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    static constexpr int LANE = 1;
};
template <> struct Opnd<1> {
    static constexpr int STEP = 32, GROUP = 1;
    typedef b8 V;
    static __device__ __forceinline__ V load(const float* p, int stride)
    {
        V v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (__bf16)p[i * stride];
        return v;
    }
    static __device__ __forceinline__ f4 mma(V a, V b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
    static constexpr int LANE = 8;
};

__device__ __forceinline__ float act_hidden(int kind, float z) { return kind == MPM_HIDDEN_RELU ? fmaxf(z, 0.f) : tanhf(z); }
// derivative of the hidden activation from its output h
__device__ __forceinline__ float dact_hidden(int kind, float h) { return kind == MPM_HIDDEN_RELU ? (h > 0.f ? 1.f : 0.f) : 1.f - h * h; }
__device__ __forceinline__ float act_out(int kind, float z) { return kind == MPM_ACT_SIGMOID ? 1.f / (1.f + expf(-z)) : z; }

__host__ __device__ __forceinline__ int pad_to(int v, int m) { return (v + m - 1) / m * m; }

// Copies rows [o0, o0 + rows) of a layer's weights (wout x win) to LDS, zero
// past the true widths, K columns (a multiple of 32), NT threads, 16 per row.
// Out-of-range elements load an element in range: loads under a condition
// would each be waited for.
template <int MW, int NT, int LD>
__device__ __forceinline__ void stage_rows(float (*dst)[LD], int rows, int K, const float* __restrict__ W, int o0, int wout,
                                           int win)
{
    constexpr int U = MW >= 64 ? 4 : 2;
    const int t = threadIdx.x & 15;
#pragma unroll 2
    for (int o = threadIdx.x >> 4; o < rows; o += NT / 16) {
        const float* row = W + (long long)min(o0 + o, wout - 1) * win;
        for (int k0 = 0; k0 < K; k0 += 16 * U) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = row[min(k0 + 16 * u + t, win - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + 16 * u + t;
                dst[o][k] = (o0 + o < wout && k < win) ? v[u] : 0.f;
            }
        }
    }
}

// Forward pass of 64 samples, 16 per wave; MW bounds the widths (32, 64 or
// 128).  What bounds it is the latency of fetching operands: read straight
// from global memory, one MFMA step waited for eight scalar loads per operand
// (BF16).  Here 64 rows of a layer's weights at a time go to LDS (68 KiB with
// the activations at 128-wide layers: two workgroups per CU), a wave's
// activations into registers once per layer, and two output tiles are formed
// at a time.  The row strides (MW + 4 words) give the 64 lanes of an operand
// read 64 different banks.  2-128-128-1, FP32, 19,897 samples: 47 us (100 with
// one workgroup per CU and a branch per step); 2-64-64-2, BF16, 32,768: 22 us;
// most of it is staging and the activations, not the matrix cores.
template <int BF16, int MW>
__global__ __launch_bounds__(256) void k_mlp_fwd(MlpDesc d, const float* __restrict__ P, long long n,
                                                 const float* __restrict__ x, float* __restrict__ y,
                                                 float* __restrict__ cache)
{
    using O = Opnd<BF16>;
    constexpr int LD = MW + 4, NS = MW / O::STEP, JB = MW < 64 ? MW : 64;
    __shared__ float s_w[JB][LD];
    __shared__ float s_a[4][16][LD];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int r = lane & 15, q = lane >> 4;
    float(*A)[LD] = s_a[w];
    const long long r0 = (long long)blockIdx.x * kRows + 16 * w;
    {
        const bool in = r0 + r < n;
        for (int k = q; k < kPad; k += 4)
            A[r][k] = (in && k < d.w[0]) ? d.in_scale[k] * x[k * n + r0 + r] + d.in_shift[k] : 0.f;
    }
    for (int l = 0; l < d.L; ++l) {
        const float* W = P + d.offW[l];
        const float* bias = P + d.offb[l];
        const int win = d.w[l], wout = d.w[l + 1];
        const int K = pad_to(win, kPad), J = pad_to(wout, kPad);
        const bool last = l == d.L - 1;
        wave_sync();
        typename O::V a[NS];
#pragma unroll
        for (int t = 0; t < NS; ++t)
            if (t * O::STEP < K) a[t] = O::load(&A[r][t * O::STEP + q * O::LANE], 1);
        wave_sync();
        for (int j0 = 0; j0 < J; j0 += JB) {
            const int rows = min(JB, J - j0);
            __syncthreads();
            stage_rows<MW, 256, LD>(s_w, rows, K, W, j0, wout, win);
            __syncthreads();
            for (int jt = 0; jt < rows; jt += 32) {
                f4 c[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                for (int g = 0; g < NS / O::GROUP; ++g)
                    if (g * O::GROUP * O::STEP < K) {
#pragma unroll
                        for (int t = g * O::GROUP; t < (g + 1) * O::GROUP; ++t) {
                            c[0] = O::mma(a[t], O::load(&s_w[jt + r][t * O::STEP + q * O::LANE], 1), c[0]);
                            c[1] = O::mma(a[t], O::load(&s_w[jt + 16 + r][t * O::STEP + q * O::LANE], 1), c[1]);
                        }
                    }
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int col = j0 + jt + 16 * e + r;
                    const float b = bias[min(col, wout - 1)];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int row = 4 * q + i;
                        float h = 0.f;
                        if (col < wout) {
                            const float z = c[e][i] + b;
                            h = last ? act_out(d.out_act, z) : act_hidden(d.hidden_act, z);
                            if (r0 + row < n) {
                                cache[d.offC[l] * n + (r0 + row) * wout + col] = h;
                                if (last) y[col * n + r0 + row] = d.shift + d.scale * h;
                            }
                        }
                        A[row][col] = h;
                    }
                }
            }
        }
    }
}

// Backward pass of 64 samples per turn, eight waves; each workgroup leaves its
// gradient of all parameters in part[blockIdx.x].  Per layer, from the last:
// dW = dZ^T H and db = column sums of dZ, then dZ of the layer below,
// dZ' = (dZ W) act'(h), which replaces H in LDS.  Weight gradients were a
// kernel of 512 samples per workgroup that fetched both operands from global
// memory, one dependent load pair per MFMA, and added to the output with
// atomics; it took three quarters of the backward pass, on a quarter of the
// CUs.  With the adjoints in LDS they are never written, and `work` holds the
// partial gradients instead.  Row stride MW + 16 words: the operand reads that
// run down the columns (four rows of 16) meet 64 different banks.
// 2-128-128-1, FP32, 19,897 samples: 67 us (146 KiB of LDS, one workgroup per
// CU, two turns for some); 2-64-64-2, BF16, 32,768: 17 us; the final sum 6-8.
// A whole training step (forward, backward, Adam): 687 -> 117 and 427 -> 47 us.
template <int BF16, int MW>
__global__ __launch_bounds__(512) void k_mlp_bwd(MlpDesc d, const float* __restrict__ P, long long n,
                                                 const float* __restrict__ x, const float* __restrict__ cache,
                                                 const float* __restrict__ dy, long long np, float* __restrict__ part)
{
    using O = Opnd<BF16>;
    constexpr int LD = MW + 16, NT = 512, NS = MW / O::STEP, GR = NT / MW;
    __shared__ float s_buf[2][kRows][LD];
    __shared__ float s_w[MW][LD];
    __shared__ float s_red[GR][MW];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = lane & 15, q = lane >> 4;
    float* out = part + (long long)blockIdx.x * np;
    const int L = d.L;
    bool first = true;
    for (long long r0 = (long long)blockIdx.x * kRows; r0 < n; r0 += (long long)gridDim.x * kRows) {
        int cur = 0;
        {
            const int wl = d.w[L], J = pad_to(wl, kPad);
            for (int i = tid; i < kRows * J; i += NT) {
                const int row = i & (kRows - 1), c = i / kRows;
                float v = 0.f;
                if (r0 + row < n && c < wl) {
                    const float h = cache[d.offC[L - 1] * n + (r0 + row) * wl + c];
                    const float g = dy[c * n + r0 + row] * d.scale;
                    v = d.out_act == MPM_ACT_SIGMOID ? g * h * (1.f - h) : g;
                }
                s_buf[0][row][c] = v;
            }
        }
        for (int l = L - 1; l >= 0; --l) {
            const int win = d.w[l], wout = d.w[l + 1];
            const int I = pad_to(win, kPad), J = pad_to(wout, kPad);
            float(*dz)[LD] = s_buf[cur];
            float(*hb)[LD] = s_buf[1 - cur];
            if (l > 0) {
                const float* hc = cache + d.offC[l - 1] * n + r0 * win;
                const float* W = P + d.offW[l];
                const int left = n - r0 < kRows ? (int)(n - r0) : kRows;
                stage_rows<MW, NT, LD>(hb, kRows, I, hc, 0, left, win);
                stage_rows<MW, NT, LD>(s_w, J, I, W, 0, wout, win);
            } else {
                for (int i = tid; i < kRows * I; i += NT) {
                    const int row = i & (kRows - 1), k = i / kRows;
                    hb[row][k] = (r0 + row < n && k < win) ? d.in_scale[k] * x[k * n + r0 + row] + d.in_shift[k] : 0.f;
                }
            }
            __syncthreads();
            // a wave keeps the operands of one tile column of H and goes down
            // every ng-th tile row of dZ
            const int ti = pad_to(win, 16) / 16, to = pad_to(wout, 16) / 16, ng = 8 / ti;
            const int i0 = (wv % ti) * 16, og = wv / ti;
            if (og < ng) {
                typename O::V bh[kRows / O::STEP];
#pragma unroll
                for (int t = 0; t < kRows / O::STEP; ++t) bh[t] = O::load(&hb[t * O::STEP + q * O::LANE][i0 + r], LD);
                for (int ot = og; ot < to; ot += ng) {
                    const int o0 = ot * 16;
                    f4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int t = 0; t < kRows / O::STEP; ++t)
                        c = O::mma(O::load(&dz[t * O::STEP + q * O::LANE][o0 + r], LD), bh[t], c);
                    const int ii = i0 + r;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int oo = o0 + 4 * q + e;
                        if (oo < wout && ii < win) {
                            float* g = &out[d.offW[l] + oo * win + ii];
                            *g = first ? c[e] : *g + c[e];
                        }
                    }
                }
            }
            {
                // column sums of dZ: GR threads per column, then one
                const int o = tid % MW, g = tid / MW;
                float sum = 0.f;
                if (o < wout)
                    for (int row = g * (kRows / GR); row < (g + 1) * (kRows / GR); ++row) sum += dz[row][o];
                s_red[g][o] = sum;
            }
            __syncthreads();
            if (tid < wout) {
                float sum = 0.f;
#pragma unroll
                for (int g = 0; g < GR; ++g) sum += s_red[g][tid];
                float* b = &out[d.offb[l] + tid];
                *b = first ? sum : *b + sum;
            }
            if (l > 0) {
                // rows 16 * (wv % 4) .. + 15, every second column tile
                const int row0 = 16 * (wv & 3);
                typename O::V a[NS];
#pragma unroll
                for (int t = 0; t < NS; ++t)
                    if (t * O::STEP < J) a[t] = O::load(&dz[row0 + r][t * O::STEP + q * O::LANE], 1);
                for (int kt = 16 * (wv >> 2); kt < I; kt += 32) {
                    f4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int g = 0; g < NS / O::GROUP; ++g)
                        if (g * O::GROUP * O::STEP < J) {
#pragma unroll
                            for (int t = g * O::GROUP; t < (g + 1) * O::GROUP; ++t)
                                c = O::mma(a[t], O::load(&s_w[t * O::STEP + q * O::LANE][kt + r], LD), c);
                        }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int row = row0 + 4 * q + i;
                        const bool in = kt + r < win && r0 + row < n;
                        hb[row][kt + r] = in ? c[i] * dact_hidden(d.hidden_act, hb[row][kt + r]) : 0.f;
                    }
                }
            }
            __syncthreads();
            cur = 1 - cur;
        }
        first = false;
    }
}

// dP = sum over the workgroups' gradients, in a fixed order: 64 parameters
// per workgroup, four waves that each sum a quarter of the parts.
__global__ __launch_bounds__(256) void k_mlp_reduce(long long np, int parts, const float* __restrict__ part,
                                                    float* __restrict__ dP)
{
    __shared__ float s[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long long i = (long long)blockIdx.x * 64 + lane;
    float sum = 0.f;
    if (i < np) {
#pragma unroll 8
        for (int b = w; b < parts; b += 4) sum += part[b * np + i];
    }
    s[w][lane] = sum;
    __syncthreads();
    if (w == 0 && i < np) dP[i] = (s[0][lane] + s[1][lane]) + (s[2][lane] + s[3][lane]);
}

__global__ void k_fill_f(float* p, long long n, float v)
{
    long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    long long stride = (long long)gridDim.x * 256;
    for (; i < n; i += stride) p[i] = v;
}

// om1 = 1 - beta1 and om2 = 1 - beta2 are formed in binary64 by the host:
// 1 - 0.999f in binary32 would carry a 1e-5 relative error.
__global__ void k_adam(long long n, float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, float lr, float b1, float b2, float om1, float om2, float eps, float c1,
                       float c2)
{
    long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float gi = g[i];
    float mi = b1 * m[i] + om1 * gi;
    float vi = b2 * v[i] + om2 * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Piecewise-constant field on an nx x ny cell grid over [lo, hi) of the first
// two coordinates; points outside take the nearest cell.
struct CellGrid {
    int nc, nx, ny;
    float lo0, lo1, inv0, inv1;
};

__device__ __forceinline__ int cell_of(const CellGrid& g, float x0, float x1)
{
    int i = (int)floorf((x0 - g.lo0) * g.inv0);
    int j = (int)floorf((x1 - g.lo1) * g.inv1);
    i = i < 0 ? 0 : (i >= g.nx ? g.nx - 1 : i);
    j = j < 0 ? 0 : (j >= g.ny ? g.ny - 1 : j);
    return j * g.nx + i;
}

__global__ void k_cell_gather(CellGrid g, long long n, const float* __restrict__ x, const float* __restrict__ table,
                              float* __restrict__ out)
{
    long long p = (long long)blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    int c = cell_of(g, x[p], x[n + p]);
    for (int k = 0; k < g.nc; ++k) out[k * n + p] = table[k * g.nx * g.ny + c];
}

// Tables past the LDS limit: one global atomic per point and component.
__global__ void k_cell_scatter(CellGrid g, long long n, const float* __restrict__ x, const float* __restrict__ dout,
                               float* __restrict__ dtable)
{
    long long p = (long long)blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    int c = cell_of(g, x[p], x[n + p]);
    for (int k = 0; k < g.nc; ++k) atomicAdd(&dtable[k * g.nx * g.ny + c], dout[k * n + p]);
}

// Table gradient summed in LDS.  A table has few entries for its points (a
// 16 x 8 table of 2 components: 14,400 points each at 1.84 M points), and
// global atomics on one address follow each other at about 140 ns: that chain
// was 2.0 ms there.  A workgroup sums its points into a binary64 copy of the
// table in LDS (ds_add_f64 runs at 4 lanes a clock, ds_add_f32 at a third of
// one) and adds it to the output once, so an address takes one global atomic
// per workgroup; a single workgroup stores its table.  `copies` (a power of
// two) tables per workgroup, taken by lane, spread the lanes of a wave that
// hit one cell; workgroups start their flush at different entries.  Gather and
// scatter together at that size: 2026 -> 26 us, of which reading and writing
// the points at the copy rate is 8.5.
constexpr int kCellBlock = 512;
constexpr int kCellPer = 4;        // points per thread and pass, loaded together
constexpr int kCellLds = 8192;     // binary64 entries of a workgroup's tables (64 KiB)
constexpr int kCellSpread = 4096;  // entries up to which a table is repeated (four workgroups of 32 KiB per CU)
constexpr int kCellWGs = 256;

// blockIdx.y = first component of the workgroup's `nk` components.
__global__ __launch_bounds__(kCellBlock) void k_cell_scatter_lds(CellGrid g, int nk, int copies, long long n,
                                                                 const float* __restrict__ x,
                                                                 const float* __restrict__ dout,
                                                                 float* __restrict__ dtable)
{
    extern __shared__ double s_tab[];
    const int cells = g.nx * g.ny, T = nk * cells, k0 = blockIdx.y * nk;
    for (int i = threadIdx.x; i < T * copies; i += kCellBlock) s_tab[i] = 0.0;
    __syncthreads();
    double* tab = s_tab + (threadIdx.x & (copies - 1)) * T;
    const long long step = (long long)gridDim.x * kCellBlock * kCellPer;
    for (long long b = (long long)blockIdx.x * kCellBlock * kCellPer + threadIdx.x; b < n; b += step) {
        float x0[kCellPer], x1[kCellPer];
#pragma unroll
        for (int q = 0; q < kCellPer; ++q) {
            const long long p = b + q * kCellBlock;
            x0[q] = p < n ? x[p] : 0.f;
            x1[q] = p < n ? x[n + p] : 0.f;
        }
        int c[kCellPer];
#pragma unroll
        for (int q = 0; q < kCellPer; ++q) c[q] = cell_of(g, x0[q], x1[q]);
        for (int k = 0; k < nk; ++k) {
            float d[kCellPer];
#pragma unroll
            for (int q = 0; q < kCellPer; ++q) {
                const long long p = b + q * kCellBlock;
                d[q] = p < n ? dout[(k0 + k) * n + p] : 0.f;
            }
#pragma unroll
            for (int q = 0; q < kCellPer; ++q)
                if (b + q * kCellBlock < n) atomicAdd(&tab[k * cells + c[q]], (double)d[q]);
        }
    }
    __syncthreads();
    const bool alone = gridDim.x == 1;
    const int at = (int)(((long long)blockIdx.x * T) / gridDim.x);
    for (int j = threadIdx.x; j < T; j += kCellBlock) {
        const int i = j + at < T ? j + at : j + at - T;
        double v = 0.0;
        for (int r = 0; r < copies; ++r) v += s_tab[r * T + i];
        float* o = &dtable[k0 * cells + i];
        if (alone) *o = (float)v;
        else if (v != 0.0) atomicAdd(o, (float)v);
    }
}

int make_cellgrid(int nc, int nx, int ny, const double* lo, const double* hi, CellGrid* g)
{
    if (nc < 1 || nx < 1 || ny < 1 || !lo || !hi || !(hi[0] > lo[0]) || !(hi[1] > lo[1])) return MPM_EINVAL;
    g->nc = nc;
    g->nx = nx;
    g->ny = ny;
    g->lo0 = (float)lo[0];
    g->lo1 = (float)lo[1];
    g->inv0 = (float)(nx / (hi[0] - lo[0]));
    g->inv1 = (float)(ny / (hi[1] - lo[1]));
    return MPM_OK;
}

int make_desc(const mpm_mlp* net, MlpDesc* d)
{
    if (!net || net->n_layers < 1 || net->n_layers > MPM_MLP_MAX_LAYERS) return MPM_EINVAL;
    if (net->math != MPM_MLP_BF16 && net->math != MPM_MLP_F32) return MPM_EINVAL;
    if (net->out_act != MPM_ACT_NONE && net->out_act != MPM_ACT_SIGMOID) return MPM_EINVAL;
    if (net->hidden_act != MPM_HIDDEN_TANH && net->hidden_act != MPM_HIDDEN_RELU) return MPM_EINVAL;
    if (net->width[0] < 1 || net->width[0] > MPM_MLP_MAX_IN) return MPM_EINVAL;
    d->L = net->n_layers;
    int off = 0;
    long long coff = 0;
    for (int l = 0; l <= d->L; ++l) {
        int wv = net->width[l];
        if (wv < 1 || wv > kMaxW) return MPM_EINVAL;
        d->w[l] = wv;
    }
    for (int l = 0; l < d->L; ++l) {
        d->offW[l] = off;
        off += d->w[l + 1] * d->w[l];
        d->offb[l] = off;
        off += d->w[l + 1];
        d->offC[l] = coff;
        coff += d->w[l + 1];
    }
    d->out_act = net->out_act;
    d->hidden_act = net->hidden_act;
    d->scale = net->out_scale;
    d->shift = net->out_shift;
    for (int k = 0; k < MPM_MLP_MAX_IN; ++k) {
        d->in_scale[k] = k < d->w[0] ? net->in_scale[k] : 0.f;
        d->in_shift[k] = k < d->w[0] ? net->in_shift[k] : 0.f;
    }
    return MPM_OK;
}

int widest(const MlpDesc& d)
{
    int m = 0;
    for (int l = 0; l <= d.L; ++l) m = d.w[l] > m ? d.w[l] : m;
    return m;
}

template <int BF16, int MW>
void launch_fwd(const MlpDesc& d, hipStream_t st, const float* P, long long n, const float* x, float* y, float* cache)
{
    k_mlp_fwd<BF16, MW><<<(unsigned)((n + kRows - 1) / kRows), 256, 0, st>>>(d, P, n, x, y, cache);
}

// `parts` workgroups, whose gradients fit the work buffer (a single one writes
// the output itself); more than the chip holds at once would only lengthen the
// final sum.
template <int BF16, int MW>
void launch_bwd(const MlpDesc& d, hipStream_t st, const float* P, long long n, const float* x, const float* cache,
                const float* dy, long long np, long long work_floats, float* work, float* dP)
{
    const long long held = MW == 128 ? 256 : 512;   // LDS: one workgroup per CU of 128-wide layers, else more
    long long parts = (n + kRows - 1) / kRows;
    parts = parts < held ? parts : held;
    parts = parts < work_floats / np ? parts : work_floats / np;
    if (parts <= 1) {
        k_mlp_bwd<BF16, MW><<<1, 512, 0, st>>>(d, P, n, x, cache, dy, np, dP);
        return;
    }
    k_mlp_bwd<BF16, MW><<<(unsigned)parts, 512, 0, st>>>(d, P, n, x, cache, dy, np, work);
    k_mlp_reduce<<<(unsigned)((np + 63) / 64), 256, 0, st>>>(np, (int)parts, work, dP);
}

}  // namespace

extern "C" {

int64_t mpm_mlp_num_params(const mpm_mlp* net)
{
    MlpDesc d;
    if (make_desc(net, &d) != MPM_OK) return -1;
    int64_t s = 0;
    for (int l = 0; l < d.L; ++l) s += (int64_t)d.w[l + 1] * (d.w[l] + 1);
    return s;
}

int64_t mpm_mlp_cache_floats(const mpm_mlp* net, int64_t n)
{
    MlpDesc d;
    if (make_desc(net, &d) != MPM_OK || n < 0) return -1;
    int64_t s = 0;
    for (int l = 1; l <= d.L; ++l) s += d.w[l];
    return s * n;
}

int mpm_mlp_forward(const mpm_mlp* net, void* hip_stream, const float* params, int64_t n, const float* x,
                    float* y, float* cache)
{
    MlpDesc d;
    int rc = make_desc(net, &d);
    if (rc) return rc;
    if (n < 0 || (n > 0 && (!params || !x || !y || !cache))) return MPM_EINVAL;
    if (n == 0) return MPM_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    const int mw = widest(d);
    if (net->math == MPM_MLP_BF16) {
        if (mw <= 32) launch_fwd<1, 32>(d, st, params, n, x, y, cache);
        else if (mw <= 64) launch_fwd<1, 64>(d, st, params, n, x, y, cache);
        else launch_fwd<1, 128>(d, st, params, n, x, y, cache);
    } else {
        if (mw <= 32) launch_fwd<0, 32>(d, st, params, n, x, y, cache);
        else if (mw <= 64) launch_fwd<0, 64>(d, st, params, n, x, y, cache);
        else launch_fwd<0, 128>(d, st, params, n, x, y, cache);
    }
    return hipGetLastError() == hipSuccess ? MPM_OK : MPM_EHIP;
}

int mpm_mlp_backward(const mpm_mlp* net, void* hip_stream, const float* params, int64_t n, const float* x,
                     const float* cache, const float* dy, float* work, float* dparams)
{
    MlpDesc d;
    int rc = make_desc(net, &d);
    if (rc) return rc;
    if (n < 0 || !dparams || (n > 0 && (!params || !x || !cache || !dy || !work))) return MPM_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    const long long np = mpm_mlp_num_params(net), wf = mpm_mlp_cache_floats(net, n);
    const int mw = widest(d);
    if (n == 0) {
        k_fill_f<<<(unsigned)((np + 255) / 256 < 1024 ? (np + 255) / 256 : 1024), 256, 0, st>>>(dparams, np, 0.f);
    } else if (net->math == MPM_MLP_BF16) {
        if (mw <= 32) launch_bwd<1, 32>(d, st, params, n, x, cache, dy, np, wf, work, dparams);
        else if (mw <= 64) launch_bwd<1, 64>(d, st, params, n, x, cache, dy, np, wf, work, dparams);
        else launch_bwd<1, 128>(d, st, params, n, x, cache, dy, np, wf, work, dparams);
    } else {
        if (mw <= 32) launch_bwd<0, 32>(d, st, params, n, x, cache, dy, np, wf, work, dparams);
        else if (mw <= 64) launch_bwd<0, 64>(d, st, params, n, x, cache, dy, np, wf, work, dparams);
        else launch_bwd<0, 128>(d, st, params, n, x, cache, dy, np, wf, work, dparams);
    }
    return hipGetLastError() == hipSuccess ? MPM_OK : MPM_EHIP;
}

int mpm_mlp_backward_noalloc(const mpm_mlp* net, void* hip_stream, const float* params, int64_t n,
                             const float* x, const float* cache, const float* dy, float* dparams)
{
    int64_t need = mpm_mlp_cache_floats(net, n);
    if (need < 0) {
        mpm::set_global_error("mpm_mlp_backward_noalloc: invalid network description or n");
        return MPM_EINVAL;
    }
    if (need > (int64_t)MPM_MLP_SCRATCH_FLOATS) {
        mpm::set_global_error("mpm_mlp_backward_noalloc: n too large for the static scratch "
                              "(mpm_mlp_cache_floats(net, n) > MPM_MLP_SCRATCH_FLOATS)");
        return MPM_EINVAL;
    }
    float* work = nullptr;
    if (n > 0) {
        int rc = scratch_address(&work);
        if (rc) return rc;
    }
    return mpm_mlp_backward(net, hip_stream, params, n, x, cache, dy, work, dparams);
}

int mpm_cell_field_gather(void* hip_stream, int32_t nc, int32_t nx, int32_t ny, const double* host_lo,
                          const double* host_hi, int64_t n, const float* x, const float* table, float* out)
{
    CellGrid g;
    if (make_cellgrid(nc, nx, ny, host_lo, host_hi, &g) || n < 0 || (n > 0 && (!x || !table || !out)))
        return MPM_EINVAL;
    if (n == 0) return MPM_OK;
    k_cell_gather<<<(unsigned)((n + 255) / 256), 256, 0, (hipStream_t)hip_stream>>>(g, n, x, table, out);
    return hipGetLastError() == hipSuccess ? MPM_OK : MPM_EHIP;
}

int mpm_cell_field_scatter(void* hip_stream, int32_t nc, int32_t nx, int32_t ny, const double* host_lo,
                           const double* host_hi, int64_t n, const float* x, const float* dout, float* dtable)
{
    CellGrid g;
    if (make_cellgrid(nc, nx, ny, host_lo, host_hi, &g) || n < 0 || !dtable || (n > 0 && (!x || !dout)))
        return MPM_EINVAL;
    hipStream_t st = (hipStream_t)hip_stream;
    const long long cells = (long long)nx * ny, nt = (long long)nc * cells;
    // all components in one table where they fit, else one at a time; few
    // points need one workgroup, which leaves nothing to clear before it
    const int nk = nt <= kCellLds ? nc : 1;
    const bool lds = cells * nk <= kCellLds && nc / nk <= 65535;
    const long long wg = (n + kCellBlock * kCellPer - 1) / (kCellBlock * kCellPer);
    const unsigned nwg = (unsigned)(wg < kCellWGs ? wg : kCellWGs);
    if (!lds || nwg != 1) k_fill_f<<<(unsigned)((nt + 255) / 256), 256, 0, st>>>(dtable, nt, 0.f);
    if (n > 0 && lds) {
        const int T = (int)(cells * nk);
        int copies = 1;
        while (copies < 16 && 2 * copies * T <= kCellSpread) copies *= 2;
        k_cell_scatter_lds<<<dim3(nwg, nc / nk), kCellBlock, (size_t)copies * T * sizeof(double), st>>>(g, nk, copies, n, x,
                                                                                                   dout, dtable);
    } else if (n > 0) {
        k_cell_scatter<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(g, n, x, dout, dtable);
    }
    return hipGetLastError() == hipSuccess ? MPM_OK : MPM_EHIP;
}

int mpm_adam_step(void* hip_stream, int64_t n, float* params, const float* grad, float* m, float* v, int32_t step,
                  double lr, double beta1, double beta2, double eps)
{
    if (n < 0 || step < 1 || (n > 0 && (!params || !grad || !m || !v))) return MPM_EINVAL;
    if (n == 0) return MPM_OK;
    float c1 = (float)(1.0 - pow(beta1, step)), c2 = (float)(1.0 - pow(beta2, step));
    k_adam<<<(unsigned)((n + 255) / 256), 256, 0, (hipStream_t)hip_stream>>>(n, params, grad, m, v, (float)lr,
                                                                              (float)beta1, (float)beta2,
                                                                              (float)(1.0 - beta1), (float)(1.0 - beta2),
                                                                              (float)eps, c1, c2);
    return hipGetLastError() == hipSuccess ? MPM_OK : MPM_EHIP;
}

}  // extern "C"
