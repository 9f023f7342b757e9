// k_gate.hip - the learned vertex-pruning gate: its inference kernel (bf16
// matrix cores, fp32 accumulation) in front of the local-moving scan, and
// the fp32 training kernels (forward, backward, Adam) of its network.
//
// Network: z = w3 . relu(W2 relu(W1 x + b1) + b2) + b3, 8 -> 64 -> 64 -> 1,
// p = sigmoid(z); a vertex is scanned iff z >= logit(theta).
//
// Inference on CDNA4 matrix cores.  A wavefront takes 64 candidates as two
// batches of 32 columns and computes the transposed layers H^T = W X^T with
// v_mfma_f32_32x32x8_bf16: operand A is a 32x8 weight tile (lane l holds row
// l%32, columns 4(l/32)..+3), operand B an 8x32 activation tile (lane l holds
// rows 4(l/32)..+3 of column l%32), and the 32x32 fp32 result leaves lane l
// with column l%32, rows 8r + 4(l/32) + q (register 4r + q).  Those rows are
// exactly the B operand of the next layer's k-step 4t + r, so the hidden
// layer goes from the accumulators to bf16 operands inside each lane: no LDS
// round trip between layers.  Per 32 columns: 2 MFMAs for layer 1, 16 for
// layer 2; the 64 -> 1 output layer is a per-lane fp32 dot product plus one
// cross-half shuffle.
#include <math.h>

#include "gsp_internal.h"

namespace gsp {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Weight operands of one lane, loaded once per wavefront.
struct NetRegs {
    s16x4 a1[2];     // W1 rows 32t + l%32, columns 4(l/32)..+3
    s16x4 a2[2][8];  // W2 rows 32t + l%32, columns 8s + 4(l/32)..+3
};

__device__ __forceinline__ void load_net(const GateNet &net, NetRegs &r) {
    const int lane = lane_id(), row = lane & 31, kq = (lane >> 5) * 4;
#pragma unroll
    for (int t = 0; t < 2; t++)
#pragma unroll
        for (int j = 0; j < 4; j++) r.a1[t][j] = (short)net.w1[(32 * t + row) * kGateFeatures + kq + j];
#pragma unroll
    for (int t = 0; t < 2; t++)
#pragma unroll
        for (int s = 0; s < 8; s++)
#pragma unroll
            for (int j = 0; j < 4; j++) r.a2[t][s][j] = (short)net.w2[(32 * t + row) * kGateHidden + 8 * s + kq + j];
}

// Logit of column l%32 of a 32-column batch whose features the lanes hold
// as B operands (bx); identical in lanes l and l^32.  The whole wavefront
// must execute this (matrix instructions need every lane).
__device__ __forceinline__ float mlp_columns(const NetRegs &r, s16x4 bx, const float *b1, const float *b2,
                                             const float *w3, float b3) {
    const int hi = lane_id() >> 5;
    f32x16 zero;
#pragma unroll
    for (int k = 0; k < 16; k++) zero[k] = 0.0f;
    s16x4 bh[8];
#pragma unroll
    for (int t = 0; t < 2; t++) {
        f32x16 c = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(r.a1[t], bx, zero, 0, 0, 0);
#pragma unroll
        for (int rr = 0; rr < 4; rr++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                int h = 32 * t + 8 * rr + 4 * hi + q;
                float v = c[4 * rr + q] + b1[h];
                v = v > 0.0f ? v : 0.0f;
                bh[4 * t + rr][q] = (short)bf16_bits(v);
            }
    }
    float part = 0.0f;
#pragma unroll
    for (int t = 0; t < 2; t++) {
        f32x16 c = zero;
#pragma unroll
        for (int s = 0; s < 8; s++) c = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(r.a2[t][s], bh[s], c, 0, 0, 0);
#pragma unroll
        for (int rr = 0; rr < 4; rr++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                int o = 32 * t + 8 * rr + 4 * hi + q;
                float v = c[4 * rr + q] + b2[o];
                v = v > 0.0f ? v : 0.0f;
                part += w3[o] * v;
            }
    }
    part += __shfl_xor(part, 32);
    return part + b3;
}

// Logits of the 64 rows fx[0..63][8] (bf16 bits) of a wavefront: the lane's
// own row's logit.
__device__ __forceinline__ float mlp_rows64(const NetRegs &r, const uint16_t (*fx)[kGateFeatures], const float *b1,
                                           const float *b2, const float *w3, float b3) {
    const int lane = lane_id(), col = lane & 31, hi = lane >> 5;
    s16x4 bx0 = *reinterpret_cast<const s16x4 *>(&fx[col][4 * hi]);
    s16x4 bx1 = *reinterpret_cast<const s16x4 *>(&fx[32 + col][4 * hi]);
    float z0 = mlp_columns(r, bx0, b1, b2, w3, b3);
    float z1 = mlp_columns(r, bx1, b1, b2, w3, b3);
    return lane < 32 ? z0 : z1;
}

__device__ __forceinline__ void load_biases(const GateNet &net, float *b1, float *b2, float *w3) {
    for (int k = threadIdx.x; k < kGateHidden; k += blockDim.x) {
        b1[k] = net.b1[k];
        b2[k] = net.b2[k];
        w3[k] = net.w3[k];
    }
}

constexpr int kGateSpan = 4096;   // candidates per workgroup, at most

// Gated sweep of one sub-round: candidates -> features -> network -> queue.
// Workgroup k takes the k-th of gridDim.x equal ranges of the candidates (at
// most kGateSpan), stages the vertices it keeps in LDS with their rank in
// their bin and reserves their queue slots with one atomic per bin.
__global__ void __launch_bounds__(kBlock) k_gate(MoveArgs a, GateNet net, float theta) {
    __shared__ float sb1[kGateHidden], sb2[kGateHidden], sw3[kGateHidden];
    __shared__ uint16_t fx[kBlock / kWave][kWave][kGateFeatures];
    __shared__ int lcnt[kNumBins], lbase[kNumBins];
    __shared__ unsigned long long spr[kBlock / kWave];
    __shared__ int32_t sv[kGateSpan];      // kept vertex
    __shared__ uint32_t sbr[kGateSpan];    // its bin (top 4 bits) and rank in the bin
    __shared__ int nst;
    load_biases(net, sb1, sb2, sw3);
    NetRegs r;
    load_net(net, r);
    int64_t pre[kNumBins + 1];
    pre[0] = 0;
#pragma unroll
    for (int b = 0; b < kNumBins; b++) pre[b + 1] = pre[b] + a.ctr->ccnt[a.round][b];
    const int64_t total = pre[kNumBins];
    int64_t span = (total + gridDim.x - 1) / gridDim.x;
    span = (span + kBlock - 1) / kBlock * kBlock;
    const int64_t lo = blockIdx.x * span;
    const int64_t hi = lo + span < total ? lo + span : total;
    const int w = threadIdx.x / kWave, lane = lane_id();
    unsigned long long pruned = 0;
    if (threadIdx.x < kNumBins) lcnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) nst = 0;
    __syncthreads();
    for (int64_t t0 = lo; t0 < hi; t0 += kBlock) {   // uniform over the workgroup
        int64_t t = t0 + threadIdx.x;
        bool valid = t < hi;
        int b = 0, i = -1;
        uint16_t x[kGateFeatures] = {0, 0, 0, 0, 0, 0, 0, 0};
        if (valid) {
            while (t >= pre[b + 1]) b++;
            i = a.cand[a.qbase[b] + (t - pre[b])];
            const int li = a.giter ? a.giter[a.g.gid[i]] : (a.iter_dev ? (int)*a.iter_dev : a.iter);
            gate_features(a.g.deg[i], a.K[i], a.sig[a.cm[i]], a.hfrac[i], a.hgain[i], a.hbits[i], a.dsnap[i], a.pass,
                          li, x);
        }
#pragma unroll
        for (int f = 0; f < kGateFeatures; f++) fx[w][lane][f] = x[f];
        __syncthreads();
        float z = mlp_rows64(r, fx[w], sb1, sb2, sw3, net.b3);
        // a batch graph outside its gated sweeps keeps every candidate
        bool keep = valid && (z >= theta || (a.ggated && !a.ggated[a.g.gid[i]]));
        if (keep) {
            const int rank = atomicAdd(&lcnt[b], 1);
            const int slot = atomicAdd(&nst, 1);
            sv[slot] = i;
            sbr[slot] = ((uint32_t)b << 28) | (uint32_t)rank;
        } else if (valid) {
            pruned++;
            if (b == BIN_HUB) a.hub_act[i] = 0;
        }
        __syncthreads();   // fx is rewritten by the next pass
    }
    if (threadIdx.x < kNumBins && lcnt[threadIdx.x] > 0)
        lbase[threadIdx.x] = atomicAdd(&a.ctr->qcnt[a.round][threadIdx.x], lcnt[threadIdx.x]);
    __syncthreads();
    for (int k = threadIdx.x; k < nst; k += kBlock) {
        const uint32_t br = sbr[k];
        const int b = (int)(br >> 28);
        a.queue[a.qbase[b] + lbase[b] + (int64_t)(br & 0x0FFFFFFFu)] = sv[k];
    }
    long long pw = group_sum_ll<kWave>((long long)pruned);
    if (lane == 0) spr[w] = (unsigned long long)pw;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long tot = 0;
        for (int q = 0; q < kBlock / kWave; q++) tot += spr[q];
        if (tot) atomicAdd(&a.ctr->st[blockIdx.x % kStripes].pruned, tot);
    }
}

// Logits of given feature rows (test hook of the inference kernel).
__global__ void __launch_bounds__(kBlock) k_gate_eval(GateNet net, const float *x, int64_t rows, float *logit) {
    __shared__ float sb1[kGateHidden], sb2[kGateHidden], sw3[kGateHidden];
    __shared__ uint16_t fx[kBlock / kWave][kWave][kGateFeatures];
    load_biases(net, sb1, sb2, sw3);
    NetRegs r;
    load_net(net, r);
    const int w = threadIdx.x / kWave, lane = lane_id();
    __syncthreads();
    for (int64_t t0 = blockIdx.x * (int64_t)kBlock; t0 < rows; t0 += (int64_t)gridDim.x * kBlock) {
        int64_t t = t0 + threadIdx.x;
#pragma unroll
        for (int f = 0; f < kGateFeatures; f++) fx[w][lane][f] = t < rows ? bf16_bits(x[t * kGateFeatures + f]) : 0;
        __syncthreads();
        float z = mlp_rows64(r, fx[w], sb1, sb2, sw3, net.b3);
        if (t < rows) logit[t] = z;
        __syncthreads();
    }
}

// ------------------------------------------------------------- training

constexpr int kR = kMlpRowsPerBlock;  // rows of one partial gradient
constexpr int kH = kGateHidden;
constexpr int kF = kGateFeatures;

__device__ __forceinline__ float softplus_f(float t) { return (t > 0.0f ? t : 0.0f) + log1pf(expf(-fabsf(t))); }
__device__ __forceinline__ float sigmoid_f(float t) {
    return t >= 0.0f ? 1.0f / (1.0f + expf(-t)) : expf(t) / (1.0f + expf(t));
}

// One training batch is three launches: k_mlp_rows (forward and backward of
// every row to the hidden layers' deltas), k_mlp_part (each block of kR rows'
// partial gradient) and k_mlp_reduce.  Every output is the same sequence of
// fp32 products and sums whatever the thread layout: a hidden unit adds its
// inputs in index order, a partial gradient its kR rows in row order, the
// reduction its blocks in block order.
//
// What bounds it: latency.  A batch of the training recipe has 4096 rows, 64
// row blocks; with a wavefront per row block (a thread per row, then a
// thread per hidden unit) 64 of the 256 CUs ran one wavefront each through
// some 12,000 multiply-adds in a row: 115 us per batch.  The rows go 16 to a
// workgroup instead (256 workgroups, 16 threads per row with four hidden
// units each: 10.1 us, of it two trips to memory for the parameters and the
// rows) and each row block's partial gradient to kPartSlices workgroups
// (5.5 us).  An epoch of 128 such batches: 17.4 -> 2.74 ms.
constexpr int kRowTile = 16;         // rows per workgroup of k_mlp_rows
constexpr int kRowThreads = 16;      // threads per row, kUnits hidden units each
constexpr int kUnits = kH / kRowThreads;
constexpr int kStride = kH + 4;      // row stride of its LDS arrays (16-byte rows)
constexpr int kPartSlices = 6;       // per row block: four quarters of W2's rows, then the other parameters
constexpr int kPartUnits = kH / (kPartSlices - 2);
static_assert(kRowTile * kRowThreads == kBlock && kUnits == 4 && kPartUnits * kH == 4 * kBlock, "thread layout");

// acts: five arrays of the slab's rows (padded to kR): h1, h2, d2, d1 with kH
// values a row, then dz; loss with one.  Rows past `rows` (the padding) run
// with x = 0 and dz = 0.
struct MlpActs {
    float *h1, *h2, *d2, *d1, *dz, *loss;
};

// acc[k] += sum over j, in order, of m[j][u0 + k] v[j].
__device__ __forceinline__ void row_times(const float (*m)[kStride], const float *v, int u0, float *acc) {
#pragma unroll 2
    for (int j = 0; j < kH; j += 8) {
        float4 w[8], x[2];
#pragma unroll
        for (int q = 0; q < 2; q++) x[q] = *reinterpret_cast<const float4 *>(v + j + 4 * q);
#pragma unroll
        for (int q = 0; q < 8; q++) w[q] = *reinterpret_cast<const float4 *>(&m[j + q][u0]);
        const float xs[8] = {x[0].x, x[0].y, x[0].z, x[0].w, x[1].x, x[1].y, x[1].z, x[1].w};
#pragma unroll
        for (int q = 0; q < 8; q++) {
            acc[0] += w[q].x * xs[q];
            acc[1] += w[q].y * xs[q];
            acc[2] += w[q].z * xs[q];
            acc[3] += w[q].w * xs[q];
        }
    }
}

__global__ void __launch_bounds__(kBlock) k_mlp_rows(const float *params, const float *x, const uint8_t *y,
                                                     int64_t rows, float pw, float inv_b, MlpActs act) {
    __shared__ __align__(16) float sW2[kH][kStride], sW2t[kH][kStride];
    __shared__ float sW1[kH][kF + 1];
    __shared__ float sb1[kH], sb2[kH];
    __shared__ __align__(16) float sw3[kH];
    __shared__ float sx[kRowTile][kF];
    __shared__ __align__(16) float sh[kRowTile][kStride], sd[kRowTile][kStride];
    __shared__ float sdz[kRowTile];
    const int tid = threadIdx.x, r = tid / kRowThreads, u0 = (tid % kRowThreads) * kUnits;
    const int64_t row = (int64_t)blockIdx.x * kRowTile + r;
    // the parameters were written by the previous launch (memory, not L2, for
    // seven of the eight XCDs): all of a thread's loads in one trip
    float w2[kH * kH / kBlock], w1[kH * kF / kBlock];
#pragma unroll
    for (int q = 0; q < kH * kH / kBlock; q++) w2[q] = params[kPW2 + q * kBlock + tid];
#pragma unroll
    for (int q = 0; q < kH * kF / kBlock; q++) w1[q] = params[kPW1 + q * kBlock + tid];
#pragma unroll
    for (int q = 0; q < kH * kH / kBlock; q++) {
        const int k = q * kBlock + tid;
        sW2[k / kH][k % kH] = w2[q];
        sW2t[k % kH][k / kH] = w2[q];
    }
#pragma unroll
    for (int q = 0; q < kH * kF / kBlock; q++) {
        const int k = q * kBlock + tid;
        sW1[k / kF][k % kF] = w1[q];
    }
    if (tid < kH) {
        sb1[tid] = params[kPB1 + tid];
        sb2[tid] = params[kPB2 + tid];
        sw3[tid] = params[kPW3 + tid];
    }
    const float b3 = params[kPB3];
    if (tid < kRowTile * kF) {
        const int64_t xr = (int64_t)blockIdx.x * kRowTile + tid / kF;
        sx[tid / kF][tid % kF] = xr < rows ? x[xr * kF + tid % kF] : 0.0f;
    }
    __syncthreads();
    float h1[kUnits], h2[kUnits], acc[kUnits];
#pragma unroll
    for (int k = 0; k < kUnits; k++) {
        float s = 0.0f;
#pragma unroll
        for (int f = 0; f < kF; f++) s += sW1[u0 + k][f] * sx[r][f];
        const float a1 = s + sb1[u0 + k];
        h1[k] = a1 > 0.0f ? a1 : 0.0f;
        sh[r][u0 + k] = h1[k];
        acc[k] = 0.0f;
    }
    __syncthreads();
    row_times(sW2t, sh[r], u0, acc);
#pragma unroll
    for (int k = 0; k < kUnits; k++) {
        const float a2 = acc[k] + sb2[u0 + k];
        h2[k] = a2 > 0.0f ? a2 : 0.0f;
        sd[r][u0 + k] = h2[k];
    }
    __syncthreads();
    if (tid < kRowTile) {   // the output unit and the loss, a thread per row
        const int64_t orow = (int64_t)blockIdx.x * kRowTile + tid;
        const bool ok = orow < rows;
        float z = 0.0f;
#pragma unroll
        for (int o = 0; o < kH; o += 4) {
            const float4 h = *reinterpret_cast<const float4 *>(&sd[tid][o]);
            const float4 w = *reinterpret_cast<const float4 *>(&sw3[o]);
            z += w.x * h.x;
            z += w.y * h.y;
            z += w.z * h.z;
            z += w.w * h.w;
        }
        z += b3;
        const float yr = ok && y[orow] ? 1.0f : 0.0f;
        float dz = 0.0f, loss = 0.0f;
        if (ok) {
            loss = pw * yr * softplus_f(-z) + (1.0f - yr) * softplus_f(z);
            dz = (sigmoid_f(z) * (pw * yr + 1.0f - yr) - pw * yr) * inv_b;
        }
        sdz[tid] = dz;
        act.dz[orow] = dz;
        act.loss[orow] = loss;
    }
    __syncthreads();
    float d2[kUnits];
    const float dz = sdz[r];
#pragma unroll
    for (int k = 0; k < kUnits; k++) {
        d2[k] = h2[k] > 0.0f ? dz * sw3[u0 + k] : 0.0f;
        sd[r][u0 + k] = d2[k];
        acc[k] = 0.0f;
    }
    __syncthreads();
    row_times(sW2, sd[r], u0, acc);
    const int64_t at = row * kH + u0;
    *reinterpret_cast<float4 *>(act.h1 + at) = make_float4(h1[0], h1[1], h1[2], h1[3]);
    *reinterpret_cast<float4 *>(act.h2 + at) = make_float4(h2[0], h2[1], h2[2], h2[3]);
    *reinterpret_cast<float4 *>(act.d2 + at) = make_float4(d2[0], d2[1], d2[2], d2[3]);
    *reinterpret_cast<float4 *>(act.d1 + at) =
        make_float4(h1[0] > 0.0f ? acc[0] : 0.0f, h1[1] > 0.0f ? acc[1] : 0.0f, h1[2] > 0.0f ? acc[2] : 0.0f,
                    h1[3] > 0.0f ? acc[3] : 0.0f);
}

// Partial gradient of row block blockIdx.x (kR rows, summed in row order) in
// the parameter layout.  Slice blockIdx.y < 4: rows [16 y, 16 y + 16) of dW2,
// thread t = hidden unit (column), group = four of those rows.  Slice 4: dW1
// and b1; slice 5: b2, w3, b3 and the block's loss, a wavefront each.
__global__ void __launch_bounds__(kBlock) k_mlp_part(const float *x, int64_t rows, float inv_b, MlpActs act,
                                                     float *part, double *part_loss) {
    __shared__ __align__(16) float sa[kR][kStride];
    __shared__ __align__(16) float sb[kR][kStride];
    __shared__ float sx[kR][kF];
    __shared__ float sz[kR], sl[kR];
    const int tid = threadIdx.x, t = tid % kH, grp = tid / kH;
    const int64_t r0 = (int64_t)blockIdx.x * kR;
    float *pp = part + (int64_t)blockIdx.x * kGateParams;
    if (blockIdx.y < kPartSlices - 2) {
        const int o0 = blockIdx.y * kPartUnits;
        for (int k = tid; k < kR * kH / 4; k += kBlock) {
            const int rr = k / (kH / 4), c = (k % (kH / 4)) * 4;
            *reinterpret_cast<float4 *>(&sa[rr][c]) = *reinterpret_cast<const float4 *>(act.h1 + (r0 + rr) * kH + c);
        }
        {
            const int rr = tid / (kPartUnits / 4), c = (tid % (kPartUnits / 4)) * 4;
            *reinterpret_cast<float4 *>(&sb[rr][c]) =
                *reinterpret_cast<const float4 *>(act.d2 + (r0 + rr) * kH + o0 + c);
        }
        __syncthreads();
        float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 16
        for (int r = 0; r < kR; r++) {
            const float hv = sa[r][t];
            const float4 d = *reinterpret_cast<const float4 *>(&sb[r][grp * 4]);
            acc[0] += d.x * hv;
            acc[1] += d.y * hv;
            acc[2] += d.z * hv;
            acc[3] += d.w * hv;
        }
#pragma unroll
        for (int k = 0; k < 4; k++) pp[kPW2 + (o0 + grp * 4 + k) * kH + t] = acc[k];
        return;
    }
    const bool first = blockIdx.y == kPartSlices - 2;
    const float *ga = first ? act.d1 : act.d2;
    for (int k = tid; k < kR * kH / 4; k += kBlock) {
        const int rr = k / (kH / 4), c = (k % (kH / 4)) * 4;
        *reinterpret_cast<float4 *>(&sa[rr][c]) = *reinterpret_cast<const float4 *>(ga + (r0 + rr) * kH + c);
        if (!first)
            *reinterpret_cast<float4 *>(&sb[rr][c]) = *reinterpret_cast<const float4 *>(act.h2 + (r0 + rr) * kH + c);
    }
    if (first) {
        for (int k = tid; k < kR * kF; k += kBlock) {
            const int64_t row = r0 + k / kF;
            sx[k / kF][k % kF] = row < rows ? x[row * kF + k % kF] : 0.0f;
        }
    } else if (tid < kR) {
        sz[tid] = act.dz[r0 + tid];
        sl[tid] = act.loss[r0 + tid];
    }
    __syncthreads();
    if (first) {
        float g[2] = {0.0f, 0.0f}, db1 = 0.0f;
#pragma unroll 16
        for (int r = 0; r < kR; r++) {
            const float d1 = sa[r][t];
            g[0] += d1 * sx[r][2 * grp];   // dW1[t][2 grp], dW1[t][2 grp + 1]
            g[1] += d1 * sx[r][2 * grp + 1];
            db1 += d1;
        }
        pp[kPW1 + t * kF + 2 * grp] = g[0];
        pp[kPW1 + t * kF + 2 * grp + 1] = g[1];
        if (grp == 0) pp[kPB1 + t] = db1;
    } else if (grp == 0) {
        float db2 = 0.0f;
#pragma unroll 16
        for (int r = 0; r < kR; r++) db2 += sa[r][t];
        pp[kPB2 + t] = db2;
    } else if (grp == 1) {
        float dw3 = 0.0f;
#pragma unroll 16
        for (int r = 0; r < kR; r++) dw3 += sz[r] * sb[r][t];
        pp[kPW3 + t] = dw3;
    } else if (grp == 2 && t == 0) {
        float db3 = 0.0f;
#pragma unroll 16
        for (int r = 0; r < kR; r++) db3 += sz[r];
        pp[kPB3] = db3;
    } else if (grp == 3 && t == 0) {
        double L = 0.0;
#pragma unroll 16
        for (int r = 0; r < kR; r++) L += (double)sl[r];
        part_loss[blockIdx.x] = L * (double)inv_b;
    }
}

// Sum of the blocks' partial gradients (in block order), then one Adam step
// (beta1 0.9, beta2 0.999, eps 1e-8) or the gradient itself.  A thread per
// parameter, kReduceAhead partials in flight at once: the sum is a serial
// chain, its loads need not be (4096-row batches, 64 partials: 19 us with the
// loads in the chain, 4.9 us with them ahead and the losses' own chain in a
// workgroup of its own).
constexpr int kReduceThreads = kWave, kReduceAhead = 64;

__global__ void __launch_bounds__(kReduceThreads) k_mlp_reduce(const float *part, const double *part_loss, int nblocks,
                                                       float *params, float *m, float *v, int adam, float lr,
                                                       float c1, float c2, float *grad, double *loss) {
    int k = blockIdx.x * kReduceThreads + threadIdx.x;
    if (k < kGateParams) {
        float g = 0.0f;
        for (int b = 0; b < nblocks; b += kReduceAhead) {
            float p[kReduceAhead];
#pragma unroll
            for (int q = 0; q < kReduceAhead; q++)
                p[q] = b + q < nblocks ? part[(int64_t)(b + q) * kGateParams + k] : 0.0f;
#pragma unroll
            for (int q = 0; q < kReduceAhead; q++)
                if (b + q < nblocks) g += p[q];
        }
        if (adam) {
            float mk = 0.9f * m[k] + 0.1f * g;
            float vk = 0.999f * v[k] + 0.001f * (g * g);
            m[k] = mk;
            v[k] = vk;
            float mh = mk / c1, vh = vk / c2;
            params[k] -= lr * mh / (sqrtf(vh) + 1e-8f);
        } else {
            grad[k] = g;
        }
    }
    if (blockIdx.x == gridDim.x - 1 && loss) {   // a workgroup of its own: the blocks' losses, in order
        double L = 0.0;
        for (int b = 0; b < nblocks; b += kReduceThreads) {
            const int m = nblocks - b < kReduceThreads ? nblocks - b : kReduceThreads;
            const double v = (int)threadIdx.x < m ? part_loss[b + threadIdx.x] : 0.0;
            for (int q = 0; q < m; q++) L += __shfl(v, q);
        }
        if (threadIdx.x == 0) *loss += L;
    }
}

inline unsigned grid_cap(int64_t units, int64_t cap) {
    if (units < 1) units = 1;
    return (unsigned)(units < cap ? units : cap);
}

}  // namespace

void launch_gate(const MoveArgs &a, const GateNet &net, float theta_logit, int64_t cap, hipStream_t s) {
    if (cap == 0) return;
    // the candidates (at most cap) are split over the grid in equal ranges of
    // at most kGateSpan
    int64_t blocks = (cap + kBlock - 1) / kBlock;
    if (blocks > 1024) blocks = 1024;
    if (blocks < (cap + kGateSpan - 1) / kGateSpan) blocks = (cap + kGateSpan - 1) / kGateSpan;
    k_gate<<<(unsigned)blocks, kBlock, 0, s>>>(a, net, theta_logit);
}

void launch_gate_eval(const GateNet &net, const float *x, int64_t rows, float *logit, hipStream_t s) {
    if (rows == 0) return;
    k_gate_eval<<<grid_cap((rows + kBlock - 1) / kBlock, 4096), kBlock, 0, s>>>(net, x, rows, logit);
}

size_t mlp_act_floats(int64_t rows) {
    if (rows > kMlpSlab) rows = kMlpSlab;
    return (size_t)((rows + kR - 1) / kR) * kR * (4 * kH + 2);
}

void launch_mlp_grad(const float *params, const float *x, const uint8_t *y, int64_t rows, float pos_weight,
                     float inv_batch, float *acts, float *part, double *part_loss, hipStream_t s) {
    for (int64_t r0 = 0; r0 < rows; r0 += kMlpSlab) {
        const int64_t len = rows - r0 < kMlpSlab ? rows - r0 : kMlpSlab, nb = (len + kR - 1) / kR, pad = nb * kR;
        MlpActs a;
        a.h1 = acts;
        a.h2 = a.h1 + pad * kH;
        a.d2 = a.h2 + pad * kH;
        a.d1 = a.d2 + pad * kH;
        a.dz = a.d1 + pad * kH;
        a.loss = a.dz + pad;
        k_mlp_rows<<<(unsigned)(pad / kRowTile), kBlock, 0, s>>>(params, x + r0 * kF, y + r0, len, pos_weight,
                                                                 inv_batch, a);
        k_mlp_part<<<dim3((unsigned)nb, kPartSlices), kBlock, 0, s>>>(x + r0 * kF, len, inv_batch, a,
                                                                      part + (r0 / kR) * kGateParams,
                                                                      part_loss + r0 / kR);
    }
}

void launch_mlp_reduce(const float *part, const double *part_loss, int nblocks, float *params, float *m, float *v,
                       bool adam, float lr, float c1, float c2, float *grad, double *loss, hipStream_t s) {
    k_mlp_reduce<<<(kGateParams + kReduceThreads - 1) / kReduceThreads + 1, kReduceThreads, 0, s>>>(part, part_loss, nblocks, params, m, v,
                                                                        adam ? 1 : 0, lr, c1, c2, grad, loss);
}

}  // namespace gsp
