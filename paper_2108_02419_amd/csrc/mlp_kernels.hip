// mlp_kernels.hip -- the surrogate network on gfx950 matrix cores: a
// 160 -> 256 -> 256 -> 256 -> 20 perceptron (ReLU, masked softmax) mapping an
// encoded in-play race state to win probabilities, trained on Monte-Carlo
// win frequencies (the frequentist estimates of paper Section 3) with a
// soft cross-entropy and Adam.
//
// Products use v_mfma_f32_16x16x32_bf16: bfloat16 operands, float32
// accumulation.  Operand fragments (one 16x32 block of A, one 32x16 block of
// B per instruction): lane l holds row / column (l % 16) and the 8
// consecutive reduction indices 8*(l/16) .. 8*(l/16)+7; the 16x16 float
// result: lane l holds column (l % 16) of rows 4*(l/16) .. 4*(l/16)+3.
//
// Fragment order: the weight copies and the activations that the weight
// gradients reduce over the batch lie in memory as the fragments are read --
// block (i, k) of 16 x 32 elements at ((i * blocks of the reduction + k) * 64
// + lane) * 8 -- so that a wave fetches one with a single contiguous 1 KB
// load.
//
// What bounds it: at the batches in use (16 to 64 rows a workgroup) not the
// products but the latency of weight fragments from L2 and of the steps
// between the layers.  So a wave fetches a whole layer's fragments before it
// needs any -- the next layer's while it finishes this one -- the softmax runs
// on half a wave a row, and a training step is three launches: forward and
// backward in one kernel with the activations kept in LDS, the weight
// gradients from fragments alone, and their sum with Adam.  Eight 2048-row
// steps and the weights read back took 786 us in seven launches a step (27 us
// forward, 20 backward, 33 weight gradients), and take 303 us so (14 forward
// and backward, 12 weight gradients, 6 Adam); 10^4 rows forward 29.3 -> 13.3.
//
// Rounding points (round to nearest even): features, weights used in
// products, hidden activations after ReLU, dz and the back-propagated
// gradients; biases, logits, probabilities, loss and weight gradients are
// float32.
#include "mlp.hpp"

namespace bbe {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float floatx4;

__device__ __forceinline__ uint16_t to_bf16(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ floatx4 mfma(bf16x8 a, bf16x8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// 16 rows x 32 reduction indices from a row-major LDS tile (stride S).
__device__ __forceinline__ bf16x8 frag_lds(const uint16_t* t, int S, int row0, int k0, int lane) {
    return *reinterpret_cast<const bf16x8*>(t + (row0 + (lane & 15)) * S + k0 + 8 * (lane >> 4));
}
// Block (i, k) of a matrix in fragment order.
__device__ __forceinline__ bf16x8 frag_ord(const uint16_t* __restrict__ m, int blocks_k, int i,
                                          int k, int lane) {
    return *reinterpret_cast<const bf16x8*>(m + ((size_t)(i * blocks_k + k) * 64 + lane) * 8);
}

constexpr int kMlpThreads = 512;     // 8 waves
constexpr int kS = kHid + 8;         // LDS row stride of hidden tiles (bank spread)
constexpr int kSin = kIn + 8;        // LDS row stride of the feature tile
constexpr int kSout = kOutP + 8;     // LDS row stride of the dz tile

// A wave's weight fragments of one layer: column blocks nb0 .. nb0 + NCB - 1.
template <int KB, int NCB>
struct Frags {
    bf16x8 b[KB][NCB];
    __device__ __forceinline__ void fetch(const uint16_t* __restrict__ w, int nb0, int lane) {
#pragma unroll
        for (int k = 0; k < KB; ++k)
#pragma unroll
            for (int c = 0; c < NCB; ++c) b[k][c] = frag_ord(w, KB, nb0 + c, k, lane);
    }
};

// acc[rb][cb] = in[16*RB x 32*KB] (LDS) * (the wave's columns).  The k blocks
// are accumulated in the same order for every row, so a row's result does not
// depend on how many rows its workgroup holds.
template <int RB, int KB, int NCB>
__device__ __forceinline__ void tile_gemm(const uint16_t* in, int S, const Frags<KB, NCB>& w,
                                          floatx4 (&acc)[RB][NCB], int lane) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[rb][cb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < KB; ++k) {
        bf16x8 a[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) a[rb] = frag_lds(in, S, rb * 16, k * 32, lane);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) acc[rb][cb] = mfma(a[rb], w.b[k][cb], acc[rb][cb]);
    }
}

// Copies rows [row0, row0 + R) of a [B][K] bf16 matrix into an LDS tile
// (stride S), zero rows past B.  16-byte pieces.
template <int R, int K>
__device__ __forceinline__ void load_tile(uint16_t* t, int S, const uint16_t* __restrict__ g,
                                          int row0, int B) {
    constexpr int P = K / 8;
    for (int i = threadIdx.x; i < R * P; i += kMlpThreads) {
        int r = i / P, c = (i - r * P) * 8;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row0 + r < B) v = *reinterpret_cast<const uint4*>(g + (size_t)(row0 + r) * K + c);
        *reinterpret_cast<uint4*>(t + r * S + c) = v;
    }
}

// Where four consecutive batch rows (rows 4*(lane/16) .. +3 of the 16 at
// `row16`) of feature column block fb go in fragment order over the batch
// (NRB blocks of 32 rows).
__device__ __forceinline__ size_t batch_place(int fb, int nrb, int row16, int lane) {
    const int g = lane >> 4;
    return ((size_t)(fb * nrb + (row16 >> 5)) * 64 + (lane & 15) +
            16 * (2 * ((row16 >> 4) & 1) + (g >> 1))) * 8 + 4 * (g & 1);
}

__device__ __forceinline__ uint2 pack4(const uint16_t (&h)[4]) {
    return make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16),
                      (uint32_t)h[2] | ((uint32_t)h[3] << 16));
}

// Hidden layer epilogue: bias, ReLU, bfloat16 into LDS (and, for training,
// in fragment order over the batch).
template <int RB, int NCB>
__device__ __forceinline__ void hidden_out(const floatx4 (&acc)[RB][NCB], int nb0,
                                           const float (&bias)[NCB], uint16_t* out,
                                           uint16_t* __restrict__ hf, int nrb, int row0,
                                           int lane) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            const int n = (nb0 + cb) * 16 + (lane & 15);
            uint16_t h[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                h[i] = to_bf16(fmaxf(acc[rb][cb][i] + bias[cb], 0.0f));
                out[(rb * 16 + 4 * (lane >> 4) + i) * kS + n] = h[i];
            }
            if (hf)
                *reinterpret_cast<uint2*>(hf + batch_place(nb0 + cb, nrb, row0 + rb * 16, lane)) =
                    pack4(h);
        }
}

// Backward-data epilogue: gradient times the ReLU mask of the forward
// activation, which it replaces in the LDS tile, and in fragment order.
template <int RB, int NCB>
__device__ __forceinline__ void grad_out(const floatx4 (&acc)[RB][NCB], int nb0, uint16_t* tile,
                                         uint16_t* __restrict__ df, int nrb, int row0,
                                         int lane) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            const int n = (nb0 + cb) * 16 + (lane & 15);
            uint16_t v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint16_t* p = tile + (rb * 16 + 4 * (lane >> 4) + i) * kS + n;
                v[i] = *p != 0 ? to_bf16(acc[rb][cb][i]) : (uint16_t)0;
                *p = v[i];
            }
            *reinterpret_cast<uint2*>(df + batch_place(nb0 + cb, nrb, row0 + rb * 16, lane)) =
                pack4(v);
        }
}

// An LDS tile of R rows (row-major, stride S, K columns) in fragment order
// over the batch: 8 rows of a column a thread.
template <int R, int K>
__device__ __forceinline__ void store_ord(const uint16_t* t, int S, uint16_t* __restrict__ f,
                                          int nrb, int row0) {
    for (int i = threadIdx.x; i < K * (R / 8); i += kMlpThreads) {
        const int c = i % K, oct = i / K;
        uint16_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = t[(oct * 8 + j) * S + c];
        const int row = row0 + oct * 8;
        const size_t at =
            ((size_t)((c >> 4) * nrb + (row >> 5)) * 64 + (c & 15) + 16 * ((row & 31) >> 3)) * 8;
        *reinterpret_cast<uint4*>(f + at) =
            make_uint4((uint32_t)v[0] | ((uint32_t)v[1] << 16),
                       (uint32_t)v[2] | ((uint32_t)v[3] << 16),
                       (uint32_t)v[4] | ((uint32_t)v[5] << 16),
                       (uint32_t)v[6] | ((uint32_t)v[7] << 16));
    }
}

// An LDS tile of hidden activations to a [B][256] matrix.
template <int R>
__device__ __forceinline__ void store_rows(const uint16_t* t, uint16_t* __restrict__ g, int row0,
                                           int B) {
    for (int i = threadIdx.x; i < R * (kHid / 8); i += kMlpThreads) {
        const int r = i / (kHid / 8), c = (i % (kHid / 8)) * 8;
        if (row0 + r < B) {
            const uint4 v = *reinterpret_cast<const uint4*>(t + r * kS + c);
            uint16_t* p = g + (size_t)(row0 + r) * kHid + c;
            // the caller's matrix may lie at any 2-byte address
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int j = 0; j < 8; ++j) p[j] = (uint16_t)(w[j >> 1] >> (16 * (j & 1)));
        }
    }
}

// Orders a wave's LDS accesses (they complete in order: this is for the
// compiler).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 20 values a row in LDS (stride kSm), summed in slot order.
constexpr int kSm = 24;
__device__ __forceinline__ float sum_slots(const float* v) {
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < kOut; ++c) s += v[c];
    return s;
}

// What the softmax needs of its rows from memory, fetched at the start of the
// kernel: half a wave a row, rows threadIdx.x / 32 + 16 * i of the tile.
template <int RB, bool kTrain>
struct RowInputs {
    int nv[RB];
    float p[RB];  // the target's slot threadIdx.x % 32 (training)
    __device__ __forceinline__ void fetch(const MlpArgs& a, int row0) {
        const int c = threadIdx.x & 31;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const int row = row0 + (int)(threadIdx.x >> 5) + 16 * i;
            nv[i] = row < a.B ? a.n_valid[row] : 1;
            if constexpr (kTrain)
                p[i] = row < a.B && c < kOut ? a.target[(size_t)row * kOut + c] : 0.0f;
        }
    }
};

// Masked softmax over the slots that hold a competitor, half a wave a row,
// lane c for slot c: probabilities, entropy, logits; for training the
// cross-entropy of each row (s_ce) and dz (into the LDS tile dz4).  Sums run
// in slot order, as one thread would form them.
template <int RB, bool kTrain>
__device__ __forceinline__ void softmax_rows(const MlpArgs& a, const RowInputs<RB, kTrain>& ri,
                                             const float (*logit)[kOutP + 1], float (*tmp)[kSm],
                                             uint16_t* dz4, float* s_ce, int row0) {
    const int c = threadIdx.x & 31;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int r = (int)(threadIdx.x >> 5) + 16 * i;
        const size_t row = (size_t)(row0 + r);
        const bool in = row0 + r < a.B;
        const int nv = min(max(ri.nv[i], 1), kOut);  // 1..20 slots hold competitors
        const bool act = c < nv;
        const float z = logit[r][c];
        float mx = act ? z : -__builtin_inff();
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        const float e = act ? expf(z - mx) : 0.0f;
        if (c < kOut) tmp[r][c] = e;
        wave_sync();
        const float sum = sum_slots(tmp[r]);
        const float inv = 1.0f / sum;
        const float q = e * inv;
        const float lq = (z - mx) - logf(sum);
        wave_sync();
        if (kTrain || a.entropy) {
            // training: the cross-entropy's terms, inference: the entropy's
            const float term = kTrain ? ri.p[i] * lq : (q > 0.0f ? q * lq : 0.0f);
            if (c < kOut) tmp[r][c] = act ? -term : 0.0f;
            wave_sync();
            const float h = sum_slots(tmp[r]);
            if (c == 0) {
                if constexpr (kTrain)
                    s_ce[r] = in ? h * a.inv_batch : 0.0f;
                else if (in)
                    a.entropy[row] = h;
            }
        }
        if constexpr (kTrain) {
            dz4[r * kSout + c] = in && act ? to_bf16((q - ri.p[i]) * a.inv_batch) : (uint16_t)0;
        } else if (in && c < kOut) {
            if (a.probs) a.probs[row * kOut + c] = q;
            if (a.logits) a.logits[row * kOutP + c] = act ? z : -__builtin_inff();
        }
    }
}

// Forward pass of 16 * RB rows; for training also the loss and the gradients
// with respect to the layers' pre-activations, with everything that the
// weight gradients need in fragment order.  Wave w: columns [32w, 32w + 32).
template <int RB, bool kTrain>
__global__ void __launch_bounds__(kMlpThreads) mlp_kernel(const MlpArgs a) {
    constexpr int R = 16 * RB;
    // inference: the layers alternate between two tiles; training keeps each
    // layer's activations until its gradient has replaced them
    constexpr int kTiles = kTrain ? 3 : 2;
    __shared__ __attribute__((aligned(16))) uint16_t s_x[R * kSin];
    __shared__ __attribute__((aligned(16))) uint16_t s_h[kTiles][R * kS];
    __shared__ float logit[R][kOutP + 1];
    __shared__ __attribute__((aligned(16))) float tmp[R][kSm];
    __shared__ __attribute__((aligned(16))) uint16_t dz4[kTrain ? R * kSout : 8];
    __shared__ float s_ce[kTrain ? R : 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row0 = blockIdx.x * R;
    const int nb0 = wave * 2;
    const int nrb = (a.B + 31) >> 5;
    uint16_t* h1 = s_h[0];
    uint16_t* h2 = s_h[1];
    uint16_t* h3 = s_h[kTrain ? 2 : 0];
    const int n = nb0 * 16 + (lane & 15);
    // With few workgroups there is nothing else on the CU to hide a fetch, so
    // fragments are fetched two layers ahead (two of the three sets of
    // registers are then in flight); otherwise one layer ahead: at 32 rows the
    // registers and 52 KB of LDS leave room for a second workgroup; at 64 rows
    // LDS (104 KB) holds one a CU, and the registers go to the accumulators.
    constexpr bool kDeep = kTrain || RB == 1;
    floatx4 acc[RB][2];
    RowInputs<RB, kTrain> ri;
    Frags<5, 2> w1;
    Frags<8, 2> w2, w3s;
    Frags<8, 2>& w3 = kDeep ? w3s : w2;
    w1.fetch(a.w1, nb0, lane);
    load_tile<R, kIn>(s_x, kSin, a.x, row0, a.B);
    if constexpr (kDeep) w2.fetch(a.w2, nb0, lane);
    if constexpr (kDeep) w3.fetch(a.w3, nb0, lane);
    ri.fetch(a, row0);
    const float b1[2] = {a.b1[n], a.b1[n + 16]};
    const float b2[2] = {a.b2[n], a.b2[n + 16]};
    const float b3[2] = {a.b3[n], a.b3[n + 16]};
    __syncthreads();
    tile_gemm<RB, 5, 2>(s_x, kSin, w1, acc, lane);
    // 32 padded outputs: two column blocks, one for each of the first waves
    Frags<8, 1> w4;
    Frags<1, 2> w4t;
    float b4 = 0.0f;
    if (wave < 2) {
        const int o = wave * 16 + (lane & 15);
        b4 = o < kOut ? a.b4[o] : 0.0f;
    }
    if constexpr (kDeep) {
        if (wave < 2) w4.fetch(a.w4, wave, lane);
        if constexpr (kTrain) w4t.fetch(a.w4t, nb0, lane);
    } else {
        w2.fetch(a.w2, nb0, lane);
    }
    hidden_out<RB, 2>(acc, nb0, b1, h1, a.hf1, nrb, row0, lane);
    if constexpr (kTrain) store_ord<R, kIn>(s_x, kSin, a.xf, nrb, row0);
    __syncthreads();
    tile_gemm<RB, 8, 2>(h1, kS, w2, acc, lane);
    if constexpr (kTrain)
        w2.fetch(a.w3t, nb0, lane);
    else if constexpr (!kDeep)
        w3.fetch(a.w3, nb0, lane);
    hidden_out<RB, 2>(acc, nb0, b2, h2, a.hf2, nrb, row0, lane);
    if constexpr (!kTrain)
        if (a.h1) store_rows<R>(h1, a.h1, row0, a.B);
    __syncthreads();
    tile_gemm<RB, 8, 2>(h2, kS, w3, acc, lane);
    if constexpr (kTrain)
        w3.fetch(a.w2t, nb0, lane);
    else if constexpr (!kDeep)
        if (wave < 2) w4.fetch(a.w4, wave, lane);
    hidden_out<RB, 2>(acc, nb0, b3, h3, a.hf3, nrb, row0, lane);
    if constexpr (!kTrain)
        if (a.h2) store_rows<R>(h2, a.h2, row0, a.B);
    __syncthreads();
    if constexpr (!kTrain)
        if (a.h3) store_rows<R>(h3, a.h3, row0, a.B);
    if (wave < 2) {
        floatx4 z[RB][1];
        tile_gemm<RB, 8, 1>(h3, kS, w4, z, lane);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                logit[rb * 16 + 4 * (lane >> 4) + i][wave * 16 + (lane & 15)] = z[rb][0][i] + b4;
    }
    __syncthreads();
    softmax_rows<RB, kTrain>(a, ri, logit, tmp, dz4, s_ce, row0);
    if constexpr (kTrain) {
        __syncthreads();
        tile_gemm<RB, 1, 2>(dz4, kSout, w4t, acc, lane);
        grad_out<RB, 2>(acc, nb0, h3, a.df3, nrb, row0, lane);
        store_ord<R, kOutP>(dz4, kSout, a.df4, nrb, row0);
        if (threadIdx.x == 0) {  // this workgroup's share of the loss, in row order
            float s = 0.0f;
            for (int r = 0; r < R; ++r) s += s_ce[r];
            a.loss_part[blockIdx.x] = s;
        }
        __syncthreads();
        tile_gemm<RB, 8, 2>(h3, kS, w2, acc, lane);
        grad_out<RB, 2>(acc, nb0, h2, a.df2, nrb, row0, lane);
        __syncthreads();
        tile_gemm<RB, 8, 2>(h2, kS, w3, acc, lane);
        grad_out<RB, 2>(acc, nb0, h1, a.df1, nrb, row0, lane);
    }
}

// Weight gradients dW[n][k] = sum over the batch rows of dz[r][n] * h[r][k],
// and bias gradients db[n] = sum over the rows of dz[r][n] (a product with a
// column of ones).  One workgroup: a 64 (n) x 64 (k) tile of one layer over
// one chunk of kWgRows rows; wave w: n rows [16w, 16w + 16) of
// the tile.  Both operands come from memory in fragment order, so there is
// nothing to stage; the tile at k0 = 0 also forms the bias gradient.  Each
// stores its tile once -- into the gradient itself when the batch is one
// chunk, else into that chunk's partial vector, and the partials are summed
// in chunk order.  No atomics, so the gradient (and training) is the same bit
// for bit from run to run.  Workgroup 0 also adds up the loss, in order.
__global__ void __launch_bounds__(256) mlp_wgrad_kernel(const MlpWgradArgs a) {
    // chunk by the low part of the workgroup's number: at 2048 rows (8 chunks)
    // each of the 8 XCDs reads one chunk of the batch
    const int chunk = blockIdx.x % a.n_parts;
    const WgradTile t = a.tiles[blockIdx.x / a.n_parts];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const LayerGrad& L = a.layers[t.layer];
    const int nrb = (a.B + 31) >> 5;
    constexpr int kRb = kWgRows / 32;
    const int rb0 = chunk * kRb;
    const int nr = min(kRb, nrb - rb0);
    if (blockIdx.x == 0 && wave == 3) {
        float s = 0.0f;
        for (int i = lane; i < a.n_loss; i += 64) s += a.loss_part[i];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) *a.loss = s;
    }
    const int nbk = (t.n0 >> 4) + wave;  // the wave's block of outputs
    if (nbk * 16 >= L.n_rows) return;
    const int kb0 = t.k0 >> 4, nkb = min(4, (L.K >> 4) - kb0);
    bf16x8 ones;
#pragma unroll
    for (int j = 0; j < 8; ++j) ones[j] = (__bf16)1.0f;
    floatx4 acc[4], accb = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[cb] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 fa[kRb], fb[kRb][4];
#pragma unroll
    for (int r = 0; r < kRb; ++r)
        if (r < nr) {
            fa[r] = frag_ord(L.dz, nrb, nbk, rb0 + r, lane);
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
                if (cb < nkb) fb[r][cb] = frag_ord(L.h, nrb, kb0 + cb, rb0 + r, lane);
        }
#pragma unroll
    for (int r = 0; r < kRb; ++r)
        if (r < nr) {
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
                if (cb < nkb) acc[cb] = mfma(fa[r], fb[r][cb], acc[cb]);
            if (t.k0 == 0) accb = mfma(fa[r], ones, accb);
        }
    const bool direct = a.n_parts == 1;
    float* out = direct ? L.gw : a.part + (size_t)chunk * kNParams + L.woff;
    float* outb = direct ? L.gb : out + L.n_rows * L.K;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int n = nbk * 16 + 4 * (lane >> 4) + i;
        if (n < L.n_rows) {
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
                if (cb < nkb) out[(size_t)n * L.K + t.k0 + cb * 16 + (lane & 15)] = acc[cb][i];
            if (t.k0 == 0 && (lane & 15) == 0) outb[n] = accb[i];
        }
    }
}

// The gradient of parameters i .. i+3: the chunks' partials in chunk order,
// chunk 0 first.
__device__ __forceinline__ float4 sum_parts(const float* __restrict__ part, int n_parts, int i) {
    float4 s = *reinterpret_cast<const float4*>(part + i);
#pragma unroll 4
    for (int c = 1; c < n_parts; ++c) {
        const float4 p = *reinterpret_cast<const float4*>(part + (size_t)c * kNParams + i);
        s.x += p.x;
        s.y += p.y;
        s.z += p.z;
        s.w += p.w;
    }
    return s;
}

__device__ __forceinline__ void store4(float* __restrict__ p, const float4& v) {
    // the caller's vector may lie at any 4-byte address
    p[0] = v.x;
    p[1] = v.y;
    p[2] = v.z;
    p[3] = v.w;
}

__global__ void __launch_bounds__(256) mlp_wreduce_kernel(const float* __restrict__ part,
                                                          int n_parts, float* __restrict__ grad) {
    const int i = 4 * (blockIdx.x * blockDim.x + threadIdx.x);
    if (i < kNParams) store4(grad + i, sum_parts(part, n_parts, i));
}

// The bfloat16 copies of W[n][k .. k+3] (K inputs, N outputs rounded up to
// 16): w in fragment order over k, wt (the transpose) over n.
__device__ __forceinline__ void copy_weights(const uint16_t (&h)[4], int n, int k, int K, int N,
                                             uint16_t* __restrict__ w,
                                             uint16_t* __restrict__ wt) {
    const size_t at =
        ((size_t)((n >> 4) * (K >> 5) + (k >> 5)) * 64 + (n & 15) + 16 * ((k & 31) >> 3)) * 8 +
        (k & 7);
    *reinterpret_cast<uint2*>(w + at) = pack4(h);
    if (wt)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            wt[((size_t)(((k + j) >> 4) * (N >> 5) + (n >> 5)) * 64 + ((k + j) & 15) +
                16 * ((n & 31) >> 3)) * 8 + (n & 7)] = h[j];
}

// Adam on the float32 master parameters (optional) and refresh of the
// bfloat16 copies used by the products; four parameters a thread (every layer
// of the packed vector starts and ends at a multiple of four).  The gradient
// is a vector, or partials to sum on the way (then also written to grad_out).
__global__ void __launch_bounds__(256) mlp_adam_kernel(const MlpAdamArgs a) {
    const int i = 4 * (blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= kNParams) return;
    float4 w = *reinterpret_cast<const float4*>(a.params + i);
    if (a.grad || a.part) {
        float4 g;
        if (a.part) {
            g = sum_parts(a.part, a.n_parts, i);
            store4(a.grad_out + i, g);
        } else {
            g = make_float4(a.grad[i], a.grad[i + 1], a.grad[i + 2], a.grad[i + 3]);
        }
        float4 m = *reinterpret_cast<const float4*>(a.m + i);
        float4 v = *reinterpret_cast<const float4*>(a.v + i);
        auto step = [&](float& w1, float& m1, float& v1, float g1) {
            m1 = a.beta1 * m1 + (1.0f - a.beta1) * g1;
            v1 = a.beta2 * v1 + (1.0f - a.beta2) * (g1 * g1);
            const float mh = m1 * a.inv_bc1;
            const float vh = v1 * a.inv_bc2;
            w1 = w1 - a.lr * mh / (sqrtf(vh) + a.eps);
        };
        step(w.x, m.x, v.x, g.x);
        step(w.y, m.y, v.y, g.y);
        step(w.z, m.z, v.z, g.z);
        step(w.w, m.w, v.w, g.w);
        *reinterpret_cast<float4*>(a.m + i) = m;
        *reinterpret_cast<float4*>(a.v + i) = v;
        *reinterpret_cast<float4*>(a.params + i) = w;
    }
    const uint16_t h[4] = {to_bf16(w.x), to_bf16(w.y), to_bf16(w.z), to_bf16(w.w)};
    // locate i in the packed layout
    if (i < kOffB1) {
        const int n = i / kIn;
        copy_weights(h, n, i - n * kIn, kIn, kHid, a.w1, nullptr);
    } else if (i >= kOffW2 && i < kOffB2) {
        const int j = i - kOffW2;
        copy_weights(h, j / kHid, j % kHid, kHid, kHid, a.w2, a.w2t);
    } else if (i >= kOffW3 && i < kOffB3) {
        const int j = i - kOffW3;
        copy_weights(h, j / kHid, j % kHid, kHid, kHid, a.w3, a.w3t);
    } else if (i >= kOffW4 && i < kOffB4) {
        const int j = i - kOffW4;
        copy_weights(h, j / kHid, j % kHid, kHid, kOutP, a.w4, a.w4t);
    }
}

// State encoding: one state per half-wave (32 lanes), lane c of the half
// for competitor c; the others' positions and times by broadcast reads of LDS
// (as 40 shuffles, and with the loads waiting for n, 10^4 states took 9.5 us
// instead of 8.6).  Slots hold competitors by expected remaining ticks
// T = (L-d) / ((lo+hi)*0.5 * (1 + rho*d/L)) (R_c taken at the midpoint of
// the remaining distance), smallest first, equal T by lower index: a
// competitor's slot is the number of competitors before it in that order.
// Early in a race that orders the field by strength, late in it by
// position.  Positions enter only relative to other competitors or to the
// line (bfloat16 keeps about 2.5 significant digits: an absolute position
// would lose the gaps that decide a race).  8 float32 features per slot,
// rounded to bfloat16: remaining distance (L-d)/L, gap to the leader /
// (75 dt), gap to the competitor directly ahead on the track (position
// order, equal positions by lower index) / (7.5 dt) capped at 4 (4 for the
// leader), previous step / (7.5 dt), mean free step (lo+hi)/(15 dt),
// (hi-lo)/(hi+lo), rho/0.2, and (T - T_min)/10; zero padding.  Each lane
// writes its slot's 8 features as one 16-byte store, so a state's 320-byte
// row is written by 20 adjacent stores.
__global__ void __launch_bounds__(256) encode_kernel(const EncodeArgs a) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    __shared__ __attribute__((aligned(16))) float tab[8][2 * kMaxN];  // (d, T) of the competitors
    const int c = threadIdx.x & 31;                // competitor of this lane
    const long b = ((long)blockIdx.x * blockDim.x + threadIdx.x) >> 5;  // state
    const bool in = b < a.B;
    const float L = a.track_len;
    // every array has 20 places a state: all are fetched at once, without
    // waiting for n
    float d = 0.0f, s = 0.0f, lo = 0.0f, hi = 0.0f, rho = 0.0f;
    int n = 0;
    if (in && c < kMaxN) {
        d = a.pos[b * kMaxN + c];
        s = a.prev[b * kMaxN + c];
        const float* cp = a.comp + (b * kMaxN + c) * 5;
        lo = cp[0];
        hi = cp[1];
        rho = cp[3];
    }
    if (in) n = min(max(a.n[b], 0), kMaxN);
    const bool act = c < n;
    const float rmid = 1.0f + rho * (d / L);
    const float T = act ? (L - d) / (((lo + hi) * 0.5f) * rmid) : __builtin_inff();
    // an empty place is behind everybody and never done
    float* row = tab[threadIdx.x >> 5];
    if (c < kMaxN) {
        row[2 * c] = act ? d : -__builtin_inff();
        row[2 * c + 1] = T;
    }
    wave_sync();
    // slot = competitors before this one in (T, index) order; the position
    // of the competitor directly ahead on the track; the leader's position;
    // the smallest expected remaining time
    int slot = 0;
    bool has_ahead = false;
    float d_above = __builtin_inff(), d_lead = -__builtin_inff(), tmin = __builtin_inff();
    auto look = [&](int i, float di, float Ti) {
        slot += (Ti < T || (Ti == T && i < c)) ? 1 : 0;
        // directly ahead: the lowest of those ahead in (position, index) order
        const bool ahead = di > d || (di == d && i < c);
        has_ahead = has_ahead || ahead;
        d_above = ahead ? fminf(d_above, di) : d_above;
        d_lead = fmaxf(d_lead, di);
        tmin = fminf(tmin, Ti);
    };
#pragma unroll
    for (int i = 0; i < kMaxN; i += 2) {
        const f32x4 q = *reinterpret_cast<const f32x4*>(row + 2 * i);
        look(i, q.x, q.y);
        look(i + 1, q.z, q.w);
    }
    if (!in || c >= kMaxN) return;
    uint16_t* x = a.x + b * kIn;
    if (act) {
        const float gap = has_ahead ? fminf((d_above - d) / a.c75, 4.0f) : 4.0f;
        const float f[8] = {(L - d) / L,     (d_lead - d) / a.c750, gap,
                            s / a.c75,       (lo + hi) / a.c15,     (hi - lo) / (hi + lo),
                            rho / 0.2f,      (T - tmin) / 10.0f};
        uint4 v;
        v.x = (uint32_t)to_bf16(f[0]) | ((uint32_t)to_bf16(f[1]) << 16);
        v.y = (uint32_t)to_bf16(f[2]) | ((uint32_t)to_bf16(f[3]) << 16);
        v.z = (uint32_t)to_bf16(f[4]) | ((uint32_t)to_bf16(f[5]) << 16);
        v.w = (uint32_t)to_bf16(f[6]) | ((uint32_t)to_bf16(f[7]) << 16);
        *reinterpret_cast<uint4*>(x + slot * 8) = v;
        if (a.slot) a.slot[b * kMaxN + slot] = c;
        if (a.target) a.target[b * kMaxN + slot] = (float)a.probs_in[b * kMaxN + c];
    } else {
        // lanes n .. 19 clear the padding slots n .. 19
        *reinterpret_cast<uint4*>(x + c * 8) = make_uint4(0u, 0u, 0u, 0u);
        if (a.slot) a.slot[b * kMaxN + c] = -1;
        if (a.target) a.target[b * kMaxN + c] = 0.0f;
    }
}

// ---------------------------------------------------------------- launchers

// Row blocks per workgroup for a batch: the most (up to 4, for training 2)
// that still give at least 256 workgroups, else 1: more rows share a fetch of
// the weights, but a CU without a workgroup costs more (10^4 rows are 313
// workgroups of 32).
static int row_blocks(int B) {
    if ((B + 63) / 64 >= 256) return 4;
    if ((B + 31) / 32 >= 256) return 2;
    return 1;
}

int mlp_train_groups(int B) { return row_blocks(B) > 1 ? (B + 31) / 32 : 2 * ((B + 31) / 32); }

hipError_t launch_mlp_fwd(const MlpArgs& a, hipStream_t s) {
    switch (row_blocks(a.B)) {
        case 4:
            hipLaunchKernelGGL((mlp_kernel<4, false>), dim3((a.B + 63) / 64), dim3(kMlpThreads), 0, s, a);
            break;
        case 2:
            hipLaunchKernelGGL((mlp_kernel<2, false>), dim3((a.B + 31) / 32), dim3(kMlpThreads), 0, s, a);
            break;
        default:
            hipLaunchKernelGGL((mlp_kernel<1, false>), dim3((a.B + 15) / 16), dim3(kMlpThreads), 0, s, a);
            break;
    }
    return hipGetLastError();
}
// Training always covers whole blocks of 32 rows (those past the batch give
// zero gradients), which the weight gradients reduce over.
hipError_t launch_mlp_train(const MlpArgs& a, hipStream_t s) {
    const int groups = mlp_train_groups(a.B);
    if (row_blocks(a.B) > 1)
        hipLaunchKernelGGL((mlp_kernel<2, true>), dim3(groups), dim3(kMlpThreads), 0, s, a);
    else
        hipLaunchKernelGGL((mlp_kernel<1, true>), dim3(groups), dim3(kMlpThreads), 0, s, a);
    return hipGetLastError();
}
hipError_t launch_mlp_wgrad(const MlpWgradArgs& a, int n_tiles, hipStream_t s) {
    hipLaunchKernelGGL(mlp_wgrad_kernel, dim3(n_tiles * a.n_parts), dim3(256), 0, s, a);
    return hipGetLastError();
}
hipError_t launch_mlp_wreduce(const float* part, int n_parts, float* grad, hipStream_t s) {
    hipLaunchKernelGGL(mlp_wreduce_kernel, dim3((kNParams / 4 + 255) / 256), dim3(256), 0, s, part,
                       n_parts, grad);
    return hipGetLastError();
}
hipError_t launch_mlp_adam(const MlpAdamArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(mlp_adam_kernel, dim3((kNParams / 4 + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}
hipError_t launch_encode(const EncodeArgs& a, hipStream_t s) {
    // 8 states per 256-thread workgroup
    hipLaunchKernelGGL(encode_kernel, dim3((unsigned)(((long)a.B + 7) / 8)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace bbe
