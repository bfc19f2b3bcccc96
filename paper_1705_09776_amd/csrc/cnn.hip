// Surrogate candidate-mask CNN on gfx950 (not from the paper: a learned gate
// in front of ALP detection).  Per image at 1/4 resolution:
//   X0 = space-to-depth(4) of u8/255 (edge-padded to a multiple of 4),
//   X_l = relu(conv3x3(X_{l-1})), l = 1..4, 16 -> 16 channels, zero padding,
//   Z = X4 . Wh + bh (16 -> 6, one logit per octave), mask bit o = Z_o > logit(tau).
// Activations are bf16 in HWC order (16 channels = 32 bytes per cell); the
// 3x3 convolutions of the forward pass and of both backward passes are bf16
// MFMAs with fp32 accumulation; the head is fp32 VALU.
//
// Parameter vector (fp32, 9382): for l = 1..4: W_l[9][16][16] ([tap][ci][co],
// tap = 3(dy+1)+(dx+1)) then b_l[16]; then Wh[16][6] ([c][o]) then bh[6].
#include "cdvs_internal.h"

namespace cdvs {

namespace {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));
// (the caller's activation and work buffers are only 8-byte aligned)
typedef short s8u __attribute__((ext_vector_type(8), aligned(8)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));

// 3x3 convolutions use v_mfma_f32_16x16x32_bf16, two taps per
// instruction: lane l holds A[l%16][8(l/16)+j] and B[8(l/16)+j][l%16] for
// j = 0..7, and D[4(l/16)+r][l%16] for r = 0..3 (checked on the device), so with k = 16 (tap - 2m) + ci the lanes
// with l/16 = 2h + c carry tap 2m + h, input channels 8c..8c+7; the tenth tap
// of the last pair is zero.
constexpr int kTapPairs = 5;
__device__ __forceinline__ f4 mfma32(const s8& a, const s8& b, const f4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0);
}

constexpr int CC = kCnnChannels;   // 16
constexpr int NHD = kCnnHeads;     // 6
constexpr int CONV_W = 9 * CC * CC;
constexpr int LAYER_P = CONV_W + CC;

// float -> bf16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ short f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (short)(u >> 16);
}
__device__ __forceinline__ float bf2f(short h) { return __uint_as_float(((uint32_t)(uint16_t)h) << 16); }
// max(x, 0) as one median (x is finite)
__device__ __forceinline__ float relu(float x) { return __builtin_amdgcn_fmed3f(x, 0.f, 3.402823466e38f); }
// Two floats -> two bf16 in one word (low half: a), by the hardware
// conversion, which rounds to nearest even as f2bf does (finite inputs).
__device__ __forceinline__ uint32_t f2bf2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f2v){a, b}, bf2v));
}

__device__ __forceinline__ int find_cell_image(const CnnImage* im, int n, int64_t cell) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (im[mid].cell0 <= cell) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Fused forward pass: the four convolutions and the head for a 32 x 16 block
// of output cells in one workgroup, with every activation kept in LDS.  For
// inference no activation goes to HBM; for training (ACTS) each layer's
// output over the block is written out as well, the same values.  (Training
// had a kernel per layer, whose waves loaded and converted all the layer's
// weights for 16 cells each, and for the first layer divided every pixel by
// 255 nine times over: 182 us for the forward pass of 614,400 cells, now
// 43 us.)  The workgroup stages the s2d input over the block
// plus a 4-cell halo (one cell per layer) and each layer writes its output
// over a region one cell smaller on every side, so the last layer covers
// exactly the block.  Cells outside the image are written as zeros at every
// layer, which is the zero padding of each convolution.
constexpr int FTW = kCnnFusedW, FTH = kCnnFusedH, FHALO = kCnnLayers;
constexpr int FFW = FTW + 2 * FHALO, FFH = FTH + 2 * FHALO;   // 40 x 24 frame
// A cell's two halves of 8 channels lie in two planes, 16 bytes per cell each:
// the 16 lanes of a B operand that read neighbouring cells' halves then read
// 256 consecutive bytes (32 bytes apart, half of them meet in a bank).  With the cells stepped on by constants instead
// of divided out, whole cells staged per lane and the head's weights read as
// scalars this took the kernel from about 179 to 151 us on 128 images of
// 640x480 (gated batch 888 -> 859 us) and from 48 to 43 us on 32 in training.
constexpr int FSTR = CC / 2;              // shorts per cell of a plane
constexpr int FPLANE = FFH * FFW * FSTR;  // shorts per plane


// MFMA weight fragments of all layers, packed once per forward call:
// frag[((l * kTapPairs + m) * 64 + lane) * 8 + j] is element j of lane
// `lane`'s A operand for tap pair m of layer l.
__global__ void k_cnn_pack(const float* __restrict__ P, short* __restrict__ frag) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kCnnLayers * kTapPairs * 64; i += gridDim.x * blockDim.x) {
        const int lane = i % 64, m = (i / 64) % kTapPairs, l = i / (64 * kTapPairs);
        const int kb = lane >> 4, t = 2 * m + (kb >> 1), c8 = (kb & 1) * 8;
        const float* Wl = P + l * LAYER_P;
#pragma unroll
        for (int j = 0; j < 8; ++j) frag[i * 8 + j] = t < 9 ? f2bf(Wl[(t * CC + c8 + j) * CC + (lane & 15)]) : (short)0;
    }
}

constexpr int FTHREADS = 512;                       // 8 waves: twice the latency hiding of 4 at the same LDS
constexpr int FSTAGE = (FFH * FFW + FTHREADS - 1) / FTHREADS;   // cells staged per lane

template <bool ACTS>
__global__ __launch_bounds__(FTHREADS, 2) void k_cnn_infer(const uint8_t* __restrict__ images, const float* __restrict__ P,
                                                      const short* __restrict__ frag,
                                                      const CnnImage* __restrict__ imgs,
                                                      const int32_t* __restrict__ owner, short* __restrict__ acts,
                                                      int64_t ncells, float* __restrict__ logits,
                                                      uint8_t* __restrict__ mask, float zthr) {
    __shared__ __align__(16) short buf[2][2 * FPLANE];
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const CnnImage g = imgs[owner[tile]];   // per-tile owner table: one load, no search
    const int lt = tile - g.ftile0;
    const int ty0 = (lt / g.ftiles_x) * FTH, tx0 = (lt % g.ftiles_x) * FTW;
    const int oy = ty0 - FHALO, ox = tx0 - FHALO;   // image cell of frame (0, 0)
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, kb = lane >> 4, li = lane & 15;
    const int H4 = g.H4, W4 = g.W4;
    // the whole frame lies inside the image (whole cells of it): no cell needs
    // a test
    const bool inside = oy >= 0 && ox >= 0 && 4 * (oy + FFH) <= g.H && 4 * (ox + FFW) <= g.W;   // uniform
    const uint8_t* img = images + g.src;
    const bool words = ((g.src | g.src_pitch | (int64_t)(uintptr_t)images) & 3) == 0;            // uniform

    // layer 0 input: s2d of the frame, zero outside the image.  A lane takes
    // whole cells (four rows of four pixels; neighbouring lanes neighbouring
    // cells); all loads are issued before the first conversion.
    uint32_t px[FSTAGE][4];
#pragma unroll
    for (int k = 0; k < FSTAGE; ++k) {
        const int it = min((int)threadIdx.x + k * FTHREADS, FFH * FFW - 1);
        const int cy = oy + it / FFW, cx = ox + it % FFW;
        if (inside && words) {
            const uint8_t* p = img + (int64_t)(4 * cy) * g.src_pitch + 4 * cx;
#pragma unroll
            for (int r = 0; r < 4; ++r) px[k][r] = *reinterpret_cast<const uint32_t*>(p + (int64_t)r * g.src_pitch);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                px[k][r] = 0;
                if (cy >= 0 && cy < H4 && cx >= 0 && cx < W4) {
                    const uint8_t* row = img + (int64_t)min(4 * cy + r, g.H - 1) * g.src_pitch;
                    const int x0 = 4 * cx;
                    if (words && x0 + 3 < g.W) {
                        px[k][r] = *reinterpret_cast<const uint32_t*>(row + x0);
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) px[k][r] |= (uint32_t)row[min(x0 + j, g.W - 1)] << (8 * j);
                    }
                }
            }
        }
    }
    const int half = kb >> 1;
    s8 a[kTapPairs];
    f4 bias;
    const s8* fr = reinterpret_cast<const s8*>(frag);
#pragma unroll
    for (int m = 0; m < kTapPairs; ++m) a[m] = fr[m * 64 + lane];
#pragma unroll
    for (int r = 0; r < 4; ++r) bias[r] = P[CONV_W + 4 * kb + r];
#pragma unroll
    for (int k = 0; k < FSTAGE; ++k) {
        const int it = threadIdx.x + k * FTHREADS;
        if (it < FFH * FFW) {
            // (u * (1 / 255) and u / 255 round to the same bf16 for every u8;
            // a cell outside the image holds zero bytes)
            uint32_t w[8];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    w[2 * r + j] = f2bf2((float)((px[k][r] >> (16 * j)) & 255u) * (1.f / 255.f),
                                         (float)((px[k][r] >> (16 * j + 8)) & 255u) * (1.f / 255.f));
            uint4* d = reinterpret_cast<uint4*>(&buf[0][it * FSTR]);
            d[0] = make_uint4(w[0], w[1], w[2], w[3]);
            d[FPLANE / 8] = make_uint4(w[4], w[5], w[6], w[7]);
        }
    }
    // (ACTS: a cell of zeros, the first of the second buffer, which no layer
    // writes: its outputs start at cell (1, 1))
    if (ACTS && threadIdx.x < 2) *reinterpret_cast<uint4*>(&buf[1][threadIdx.x * FPLANE]) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();

    // The layers are unrolled, so each layer's output region is a constant.  A
    // lane's cell is stepped on by constants from one pair of 16-cell groups
    // to the wave's next, with its offset in a plane; the B operand of tap
    // pair m is read at one of three per-lane bases plus a constant: tap 0 of
    // the cell (the cell at (-1, -1)), shifted for the lanes that carry the
    // pair's second tap by that tap's distance from the first, which is one
    // cell for pairs 0, 2 and 3 and FFW - 2 cells for pair 1.  Pair 4's second
    // tap is zero in the A operand: for training its lanes read the cell of
    // zeros (an activation that has become infinite would give 0 x inf there,
    // where the backward pass has to see what the nine taps give), for
    // inference tap 8's cell again.  All ten loads of a step are issued before
    // its MFMAs.
    constexpr int CB = FSTR * 2;            // bytes per cell of a plane
    constexpr int STEP = 32 * (FTHREADS / 64);
#pragma unroll
    for (int l = 0; l < kCnnLayers; ++l) {
        // the next layer's fragments load while this layer computes
        s8 an[kTapPairs];
        f4 bn;
        const int ln = l + 1 < kCnnLayers ? l + 1 : l;
#pragma unroll
        for (int m = 0; m < kTapPairs; ++m) an[m] = fr[(ln * kTapPairs + m) * 64 + lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) bn[r] = P[ln * LAYER_P + CONV_W + 4 * kb + r];
        const char* X = reinterpret_cast<const char*>(buf[l & 1]) + (kb & 1) * (FPLANE * 2);
        const char* Z = reinterpret_cast<const char*>(buf[1]) + (kb & 1) * (FPLANE * 2);
        const char* XA = X + half * CB;
        const char* XB = X + half * (FFW - 2) * CB;
        char* Y = reinterpret_cast<char*>(buf[(l + 1) & 1]) + half * (FPLANE * 2) + 8 * (kb & 1) + (FFW + 1) * CB;
        const int lo = l + 1, C = FFW - 2 * lo, n = (FFH - 2 * lo) * C;
        // tap t = 3 (dy + 1) + (dx + 1) at byte offset (dy + 1) FFW CB + (dx + 1) CB from tap 0
        auto toff = [](int t) { return ((t / 3) * FFW + t % 3) * CB; };
        int fy[2], fx[2], off[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int q = min(wave * 32 + 16 * h + li, n - 1);
            fy[h] = lo + q / C;
            fx[h] = lo + q % C;
            off[h] = ((fy[h] - 1) * FFW + fx[h] - 1) * CB;
        }
        for (int q0 = wave * 32; q0 < n; q0 += STEP) {
            s8 b[kTapPairs][2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // (past the region's end: its last cell again, not written)
                const int o = min(off[h], ((FFH - lo - 2) * FFW + FFW - lo - 2) * CB);
                b[0][h] = *reinterpret_cast<const s8*>(XA + o + toff(0));
                b[1][h] = *reinterpret_cast<const s8*>(XB + o + toff(2));
                b[2][h] = *reinterpret_cast<const s8*>(XA + o + toff(4));
                b[3][h] = *reinterpret_cast<const s8*>(XA + o + toff(6));
                b[4][h] = *reinterpret_cast<const s8*>(ACTS && half ? Z : X + o + toff(8));
            }
            f4 acc[2] = {bias, bias};
#pragma unroll
            for (int m = 0; m < kTapPairs; ++m)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    // (the tenth tap's products add exact zeros: its A fragment
                    // is zero and the activations are finite and non-negative)
                    acc[h] = mfma32(a[m], b[m][h], acc[h]);
                }
            // relu, bf16, zero outside the image (selected, no branch), one
            // 8-byte store per cell.  Both groups' values are settled before
            // the first store: a uniform branch right behind the MFMAs was
            // compiled with 7 wait states up to the first read of their result on
            // its taken side, where straight-line code gets 8, and read old values.
            uint2 o[2];
            bool in[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                in[h] = (unsigned)(oy + fy[h]) < (unsigned)H4 && (unsigned)(ox + fx[h]) < (unsigned)W4;
                o[h].x = f2bf2(relu(acc[h][0]), relu(acc[h][1]));
                o[h].y = f2bf2(relu(acc[h][2]), relu(acc[h][3]));
                o[h].x = in[h] ? o[h].x : 0u;
                o[h].y = in[h] ? o[h].y : 0u;
            }
            asm volatile("" : "+v"(o[0].x), "+v"(o[0].y), "+v"(o[1].x), "+v"(o[1].y));
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (q0 + 16 * h + li < n) {
                    *reinterpret_cast<uint2*>(Y + off[h]) = o[h];
                    // the block's own cells also go out for the backward pass
                    if (ACTS && in[h] && (unsigned)(fy[h] - FHALO) < (unsigned)FTH && (unsigned)(fx[h] - FHALO) < (unsigned)FTW)
                        *reinterpret_cast<uint2*>(acts + ((int64_t)l * ncells + g.cell0 +
                                                          (int64_t)(oy + fy[h]) * W4 + ox + fx[h]) * CC + 4 * kb) = o[h];
                }
                // the wave's next group
                fx[h] += STEP % C;
                fy[h] += STEP / C;
                const bool wrap = fx[h] >= lo + C;
                off[h] += (STEP / C * FFW + STEP % C) * CB + (wrap ? (FFW - C) * CB : 0);
                fx[h] -= wrap ? C : 0;
                fy[h] += wrap ? 1 : 0;
            }
        }
#pragma unroll
        for (int m = 0; m < kTapPairs; ++m) a[m] = an[m];
        bias = bn;
        __syncthreads();
    }

    // head on the last layer's output (kCnnLayers is even: it is in buf[0]),
    // one cell per lane; the weights are the same for every lane
    static_assert(FTH * FTW == FTHREADS, "one cell per lane");
    const int hy = threadIdx.x / FTW, hx = threadIdx.x % FTW;
    if (ty0 + hy >= H4 || tx0 + hx >= W4) return;
    const uint4* xs = reinterpret_cast<const uint4*>(&buf[kCnnLayers & 1][((FHALO + hy) * FFW + FHALO + hx) * FSTR]);
    const uint4 xa = xs[0], xb = xs[FPLANE / 8];
    const uint32_t xw[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
    const float* Wh = P + kCnnLayers * LAYER_P;
    const int64_t c = g.cell0 + (int64_t)(ty0 + hy) * W4 + tx0 + hx;
    uint32_t bits = 0;
#pragma unroll
    for (int o = 0; o < NHD; ++o) {
        float z = Wh[CC * NHD + o];
#pragma unroll
        for (int ch = 0; ch < CC; ++ch)
            z = fmaf(__uint_as_float(ch & 1 ? xw[ch / 2] & 0xFFFF0000u : xw[ch / 2] << 16), Wh[ch * NHD + o], z);
        if (logits) logits[c * NHD + o] = z;
        if (o < g.n_oct && z > zthr) bits |= 1u << o;
    }
    if (mask) mask[c] = (uint8_t)bits;
}

__device__ __forceinline__ float softplus(float z) { return fmaxf(z, 0.f) + log1pf(expf(-fabsf(z))); }

// Sums, over the 64 lanes of the wave, of N values per lane (N a power of
// two, at most 64): at each distance a lane hands over the half of its values
// that its partner keeps, so the values halve as the lanes they cover double
// (N - 1 exchanges in all, against 6 N for a butterfly of each value); lane l
// returns the sum of value l % N.
template <int N>
__device__ __forceinline__ float wave_sums(float (&v)[N], int lane) {
    if constexpr (N > 1) {
        float h[N / 2];
        const bool up = (lane & (N / 2)) != 0;
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            const float keep = up ? v[i + N / 2] : v[i], send = up ? v[i] : v[i + N / 2];
            h[i] = keep + __uint_as_float(lane_xor<N / 2>(__float_as_uint(send)));
        }
        return wave_sums<N / 2>(h, lane);
    } else {
        return v[0];
    }
}

// The first `n` words of out[] (the last in out_last when that is not null)
// as the sums of `parts` rows of `stride` floats: 32 columns per workgroup
// (the block-th), whose 32 lane rows take every 32nd row each.  The rows are
// large against their sum (gradients cancel), so they are added in 64 bits, at
// no cost in a launch that waits for its loads (training step of 32 images
// 154.7 us either way; the four waves' sums of k_conv_bwd too: 156.9).
constexpr int kSumCols = 32, kSumRows = 32;
__device__ __forceinline__ void sum_parts(int block, const float* __restrict__ part, int parts, int stride, int n,
                                          float* __restrict__ out, float* __restrict__ out_last) {
    __shared__ double red[kSumRows][kSumCols + 1];
    const int c = threadIdx.x % kSumCols, r = threadIdx.x / kSumCols, col = block * kSumCols + c;
    double s = 0.0;
    if (col < n) {
#pragma unroll 4
        for (int p = r; p < parts; p += kSumRows) s += (double)part[(int64_t)p * stride + col];
    }
    red[r][c] = s;
    __syncthreads();
    if (r == 0 && col < n) {
#pragma unroll
        for (int i = 1; i < kSumRows; ++i) s += red[i][c];
        if (out_last && col == n - 1) *out_last = (float)s;
        else out[col] = (float)s;
    }
}

// Head backward + loss: per cell dZ, the masked gradient dP4 = (dZ Wh^T) *
// (X4 > 0) as bf16, and the sums of dWh, dbh and the loss over this
// workgroup's cells as one row of `part` (k_sum_all adds the rows).  The
// loss is the mean over images of each image's mean over cells and its
// octaves.
//
// 64 B read and 32 B written per cell would take 9 us for 614,400 cells at a
// copy's rate; what bounds it is the issue of the six exponentials, logarithms
// and divisions per cell at two waves per SIMD.  Each lane sums its
// own cells' 103 products in registers; adding them up used to take 6
// exchanges per value and one global atomic per value and wave, all on the
// same 7 cache lines, which was nearly all of the kernel's time (931 us for
// 614,400 cells); with the halving exchange, one row of sums per workgroup
// and no atomics it took 34 us.  Two waves per SIMD (the
// sums take the registers) hide little: with the next cell's values fetched
// ahead, no image lookup per cell, and dZ Wh^T as 24 matrix instructions
// instead of 96 FMAs with spilled scalar weights it takes 28.
constexpr int kHeadSums = CC * NHD + NHD + 1;   // dWh, dbh, loss: 103
constexpr int kHeadRow = 104;                   // floats per row of sums
__global__ __launch_bounds__(256) void k_head_bwd(const short* __restrict__ X4, const float* __restrict__ P,
                                                  const float* __restrict__ logits, const uint32_t* __restrict__ labels,
                                                  const float* __restrict__ pos_w, const CnnImage* __restrict__ imgs,
                                                  int nimg, int64_t ncells, int per_block, short* __restrict__ dP4,
                                                  float* __restrict__ part) {
    __shared__ float red[4][128];
    const float* Wh = P + kCnnLayers * LAYER_P;
    // A operands: the lane's weight, channel 4 q + (lane & 3) to head o
    float wa[CC / 4][NHD];
#pragma unroll
    for (int q = 0; q < CC / 4; ++q)
#pragma unroll
        for (int o = 0; o < NHD; ++o) wa[q][o] = Wh[(4 * q + (threadIdx.x & 3)) * NHD + o];
    // values 0..95: dWh[channel][head]; 96..101: dbh; 102: loss; the rest 0
    float g0[64], g1[64];
#pragma unroll
    for (int i = 0; i < 64; ++i) g0[i] = g1[i] = 0.f;
    auto add = [&](int i, float v) {
        if (i < 64) g0[i] += v;
        else g1[i - 64] += v;
    };
    // a contiguous range of cells per workgroup: its first cell's image is
    // searched for once (the same for all lanes), and a lane reads the next
    // one's entry only where its cells reach it
    const int64_t beg = (int64_t)blockIdx.x * per_block, end = min(beg + per_block, ncells);
    int64_t c = beg + threadIdx.x;
    int im = find_cell_image(imgs, nimg, beg), n_oct;
    int64_t next_cell0;   // where the next image starts
    float scale;
    auto enter = [&]() {
        const CnnImage& g = imgs[im];
        n_oct = g.n_oct;
        scale = 1.f / ((float)g.H4 * (float)g.W4 * (float)n_oct * (float)nimg);
        next_cell0 = im + 1 < nimg ? imgs[im + 1].cell0 : ncells;
    };
    enter();
    // (the next cell's values are on the way while this one's are used)
    s8 na{}, nb{};
    float nz[NHD] = {};
    uint32_t ny = 0u;
    auto fetch = [&](int64_t cell) {
        const s8u* xp = reinterpret_cast<const s8u*>(X4 + cell * CC);
        na = xp[0];
        nb = xp[1];
#pragma unroll
        for (int o = 0; o < NHD; ++o) nz[o] = logits[cell * NHD + o];
        ny = labels[cell];
    };
    if (c < end) fetch(c);
    for (int64_t c0 = beg; c0 < end; c0 += blockDim.x, c += blockDim.x) {   // uniform: matrix instructions run on whole waves
        const bool in = c < end;
        while (in && c >= next_cell0) {
            ++im;
            enter();
        }
        const uint32_t y = ny;
        const s8 xa = na, xb = nb;
        float zc[NHD];
#pragma unroll
        for (int o = 0; o < NHD; ++o) zc[o] = nz[o];
        if (c + blockDim.x < end) fetch(c + blockDim.x);
        float dz[NHD];
#pragma unroll
        for (int o = 0; o < NHD; ++o) {
            const float z = zc[o];
            const float yo = (float)((y >> o) & 1u), w = pos_w[o];
            const float s = 1.f / (1.f + expf(-z));
            const bool on = in && o < n_oct;
            dz[o] = on ? (s * (w * yo + 1.f - yo) - w * yo) * scale : 0.f;
            add(102, on ? (w * yo * softplus(-z) + (1.f - yo) * softplus(z)) * scale : 0.f);
            add(96 + o, dz[o]);
        }
        s8 oa, ob;
        // dZ Wh^T: step o of the 4x4x1 products adds head o's dZ of the lane's
        // cell times its weights to four channels at a time, each product
        // rounded as an fma, so the same chain as fma(Wh, dz, d) over o
        f4 dq[CC / 4];
#pragma unroll
        for (int q = 0; q < CC / 4; ++q) dq[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int o = 0; o < NHD; ++o)
#pragma unroll
            for (int q = 0; q < CC / 4; ++q) dq[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(wa[q][o], dz[o], dq[q], 0, 0, 0);
#pragma unroll
        for (int ch = 0; ch < CC; ++ch) {
            const float x = bf2f(ch < 8 ? xa[ch] : xb[ch - 8]);
            const float d = dq[ch / 4][ch % 4];
#pragma unroll
            for (int o = 0; o < NHD; ++o) {
                const int i = ch * NHD + o;
                if (i < 64) g0[i] = fmaf(x, dz[o], g0[i]);
                else g1[i - 64] = fmaf(x, dz[o], g1[i - 64]);
            }
            const short v = f2bf(x > 0.f ? d : 0.f);
            if (ch < 8) oa[ch] = v;
            else ob[ch - 8] = v;
        }
        if (in) {
            s8u* dst = reinterpret_cast<s8u*>(dP4 + c * CC);
            dst[0] = oa;
            dst[1] = ob;
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    red[wave][lane] = wave_sums(g0, lane);
    red[wave][64 + lane] = wave_sums(g1, lane);
    __syncthreads();
    const int t = threadIdx.x;
    if (t < kHeadSums) part[(int64_t)blockIdx.x * kHeadRow + t] = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
}

// Backward of layer l: the weight and bias gradients
// dW[t][ci][co] = sum_p X_{l-1}[p + d_t][ci] dP_l[p][co], db[co] = sum_p dP_l[p][co],
// as v_mfma_f32_16x16x32_bf16 with K = 32 cells of one row, and, but for the
// first layer, the input gradient dX_{l-1}[p][ci] = sum_t sum_co W[t][ci][co]
// dP_l[p - d_t][co], times (X_{l-1} > 0) to give dP_{l-1} (bf16).
//
// One 256-lane workgroup per tile of 32 x 16 cells at a time, the grid
// striding over the tiles with the sums kept in registers.  Both operands
// need their cells along K, while a cell's 16 channels are contiguous in
// memory: the tile of dP and the tile of X with a one-cell rim are staged
// through LDS transposed ([row][channel][cell], two cells packed per 4-byte
// write; row strides of 40 and 56 shorts put the 16 channels of an operand
// read on different banks).  A wave takes four rows: a row of X is read once
// and, shifted by a cell either way in registers, serves the nine taps of up
// to three rows of dP.  The workgroup's four waves are added up in LDS and
// written as one row of sums for k_sum_all.
//
// The input gradient's operand has its channels along K: the tile of dP with
// its rim lies in LDS a second time, as in memory (19 KB), and each wave
// gives the four rows that it has just summed.  One tap per
// v_mfma_f32_16x16x16_bf16 (lane l holds A[l%16][4(l/16)+j] and
// B[4(l/16)+j][l%16] for j = 0..3), in the order of the taps: two taps per
// instruction add up in another order, whose roundings to bf16 an Adam step
// then carries on.
//
// Bound by the latency of a tile's loads and transposes at two workgroups
// per CU; 96 B per cell are needed (64 in the first layer), 12 us.  For
// 614,400 cells: gathering operands two bytes at a time, adding every wave's
// sums with global atomics, and a wave per 16 cells converting all the
// weights for itself took 272 + 41 us (303 in the first layer, which also
// divided per pixel); one launch for the weights and one for the inputs, each
// with tiles of its own, 13 + 13; the two on one tile 22.  The first layer,
// whose loads are eight rows of pixels, has its next tile's out before it
// works on this one: 17 -> 14.5; the others gain nothing by it and lose 1 us
// where a workgroup has one tile.  The tiles go round the XCDs as they come:
// neighbours on one XCD gave 23.
constexpr int WTW = kCnnFusedW, WTH = kCnnFusedH;   // 32 x 16 cells
constexpr int WXS = 56, WPS = 40;                   // LDS strides of a channel's row of X and dP (shorts)
constexpr int WX0 = 8;                              // position of the tile's first cell in a row of X
constexpr int kConvSums = LAYER_P;                  // dW (9 x 16 x 16), db (16)
static_assert(WTW == 32 && WTH == 16, "a wave takes four rows of 32 cells");

// What 8 channels (8 half ..) of cell (cy, cx) of the layer input are made
// of: their 16 bytes, or the two rows of four pixels of the space-to-depth
// image when FIRST; zero outside the image.
template <bool FIRST>
struct Cell8 {
    using type = s8;
};
template <>
struct Cell8<true> {
    using type = uint2;
};

template <bool FIRST>
__device__ __forceinline__ typename Cell8<FIRST>::type load_cell8(const uint8_t* __restrict__ images,
                                                                  const short* __restrict__ X, const CnnImage& g, int cy,
                                                                  int cx, int half) {
    typename Cell8<FIRST>::type v = {};
    if (cy < 0 || cy >= g.H4 || cx < 0 || cx >= g.W4) return v;
    if constexpr (!FIRST) {
        v = *reinterpret_cast<const s8u*>(X + (g.cell0 + (int64_t)cy * g.W4 + cx) * CC + 8 * half);
    } else {
        uint32_t px[2] = {0, 0};
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const uint8_t* row = images + g.src + (int64_t)min(4 * cy + 2 * half + r, g.H - 1) * g.src_pitch;
            const int x0 = 4 * cx;
            if (x0 + 3 < g.W && ((uintptr_t)(row + x0) & 3) == 0) {
                px[r] = *reinterpret_cast<const uint32_t*>(row + x0);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) px[r] |= (uint32_t)row[min(x0 + j, g.W - 1)] << (8 * j);
            }
        }
        v = make_uint2(px[0], px[1]);
    }
    return v;
}

__device__ __forceinline__ s8 cell8_bf16(s8 v) { return v; }
__device__ __forceinline__ s8 cell8_bf16(uint2 v) {
    s8 o;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const uint32_t px = r == 0 ? v.x : v.y;
        // u * (1 / 255) and u / 255 round to the same bf16 for every u8
        const float k = 1.f / 255.f;
        const uint32_t lo = f2bf2((float)(px & 255u) * k, (float)((px >> 8) & 255u) * k);
        const uint32_t hi = f2bf2((float)((px >> 16) & 255u) * k, (float)(px >> 24) * k);
        o[4 * r] = (short)lo;
        o[4 * r + 1] = (short)(lo >> 16);
        o[4 * r + 2] = (short)hi;
        o[4 * r + 3] = (short)(hi >> 16);
    }
    return o;
}

template <bool FIRST>
__global__ __launch_bounds__(256, 2) void k_conv_bwd(const uint8_t* __restrict__ images, const short* __restrict__ Xprev,
                                                     const short* __restrict__ dP, const float* __restrict__ Wl,
                                                     const CnnImage* __restrict__ imgs, const int32_t* __restrict__ owner,
                                                     int ntiles, float* __restrict__ part, short* __restrict__ dPprev) {
    constexpr int XP = WTW / 2 + 2;                      // cell pairs per staged row of X: cells -2 .. 33
    constexpr int NX = (WTH + 2) * XP * 2, NP = WTH * (WTW / 2) * 2;
    constexpr int JX = (NX + 255) / 256, JP = NP / 256;
    static_assert(NP % 256 == 0, "whole rounds");
    __shared__ __align__(16) short Xt[(WTH + 2) * CC * WXS];
    __shared__ __align__(16) short Pt[WTH * CC * WPS];
    // the tile of dP with its rim, as it lies in memory (input gradients only)
    constexpr int PW = WTW + 2, PH = WTH + 2, NB = FIRST ? 0 : 2 * (PW * PH - WTW * WTH);
    static_assert(NB <= 256, "the rim in one round");
    __shared__ __align__(16) short buf[FIRST ? 8 : PH * PW * CC];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, kb = lane >> 4, li = lane & 15;
    f4 acc[9], accb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
    const short one = 0x3F80;   // 1.0: a row of ones sums dP itself
    const s8 ones = {one, one, one, one, one, one, one, one};
    s4 wt[9];   // A[ci = lane % 16][co]
    if constexpr (!FIRST) {
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const float* w = Wl + (t * CC + li) * CC + 4 * kb;
            wt[t] = __builtin_bit_cast(s4, make_uint2(f2bf2(w[0], w[1]), f2bf2(w[2], w[3])));
        }
    }
    // this thread's half cell of the rim: the top and bottom rows, then the sides
    const int rim = tid >> 1, side = rim - 2 * PW;
    const int rim_r = rim < 2 * PW ? (rim < PW ? 0 : PH - 1) : 1 + (side >> 1);
    const int rim_c = rim < 2 * PW ? (rim < PW ? rim : rim - PW) : (side & 1) * (PW - 1);
    uint32_t* X32 = reinterpret_cast<uint32_t*>(Xt);
    uint32_t* P32 = reinterpret_cast<uint32_t*>(Pt);
    // Every load of a tile goes out before its first LDS write; an item is
    // half of the channels of two neighbouring cells.
    CnnImage g;
    int ty0, tx0;
    typename Cell8<FIRST>::type xv[JX][2];
    s8 pv[JP][2], bv = {0, 0, 0, 0, 0, 0, 0, 0};
    auto fetch = [&](int tile) {
        g = imgs[owner[tile]];
        const int lt = tile - g.ftile0;
        ty0 = (lt / g.ftiles_x) * WTH;
        tx0 = (lt % g.ftiles_x) * WTW;
#pragma unroll
        for (int j = 0; j < JX; ++j) {
            const int it = tid + 256 * j, half = it & 1, k = (it >> 1) % XP, r = (it >> 1) / XP;
#pragma unroll
            for (int c = 0; c < 2; ++c)
                xv[j][c] = load_cell8<FIRST>(images, Xprev, g, it < NX ? ty0 - 1 + r : -1, tx0 - 2 + 2 * k + c, half);
        }
#pragma unroll
        for (int j = 0; j < JP; ++j) {
            const int it = tid + 256 * j, half = it & 1, k = (it >> 1) % (WTW / 2), r = (it >> 1) / (WTW / 2);
#pragma unroll
            for (int c = 0; c < 2; ++c) pv[j][c] = load_cell8<false>(nullptr, dP, g, ty0 + r, tx0 + 2 * k + c, half);
        }
        if constexpr (!FIRST) bv = load_cell8<false>(nullptr, dP, g, tid < NB ? ty0 - 1 + rim_r : -1, tx0 - 1 + rim_c, tid & 1);
    };
    if (FIRST && (int)blockIdx.x < ntiles) fetch(blockIdx.x);
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        if (!FIRST) fetch(tile);
        __syncthreads();   // the previous tile's readers are done
#pragma unroll
        for (int j = 0; j < JX; ++j) {
            const int it = tid + 256 * j, half = it & 1, k = (it >> 1) % XP, r = (it >> 1) / XP;
            if (it < NX) {
                const s8 x0 = cell8_bf16(xv[j][0]), x1 = cell8_bf16(xv[j][1]);
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    X32[((r * CC + 8 * half + c) * WXS + WX0 - 2) / 2 + k] =
                        (uint32_t)(uint16_t)x0[c] | ((uint32_t)(uint16_t)x1[c] << 16);
            }
        }
#pragma unroll
        for (int j = 0; j < JP; ++j) {
            const int it = tid + 256 * j, half = it & 1, k = (it >> 1) % (WTW / 2), r = (it >> 1) / (WTW / 2);
#pragma unroll
            for (int c = 0; c < 8; ++c)
                P32[(r * CC + 8 * half + c) * WPS / 2 + k] =
                    (uint32_t)(uint16_t)pv[j][0][c] | ((uint32_t)(uint16_t)pv[j][1][c] << 16);
            if constexpr (!FIRST) {
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    reinterpret_cast<s8*>(buf)[((r + 1) * PW + 2 * k + c + 1) * 2 + half] = pv[j][c];
            }
        }
        if constexpr (!FIRST) {
            if (tid < NB) reinterpret_cast<s8*>(buf)[(rim_r * PW + rim_c) * 2 + (tid & 1)] = bv;
        }
        // the rows' own activations, needed only for the input gradients
        s4 xp[4][2];
        const int cy0 = ty0 + 4 * wave, cx0 = tx0 + li, H4 = g.H4, W4 = g.W4;
        const int64_t off0 = (g.cell0 + (int64_t)cy0 * W4 + cx0) * CC + 4 * kb;
        if constexpr (!FIRST) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    xp[q][h] = s4{0, 0, 0, 0};
                    if (cy0 + q < H4 && cx0 + 16 * h < W4)
                        xp[q][h] = *reinterpret_cast<const s4*>(Xprev + off0 + (int64_t)(q * W4 + 16 * h) * CC);
                }
        }
        __syncthreads();
        if (FIRST && tile + (int)gridDim.x < ntiles) fetch(tile + gridDim.x);
        // this wave's rows of dP: 4 wave .. 4 wave + 3; B[k = cell 8 kb + j][co = li]
        s8 b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            b[q] = *reinterpret_cast<const s8*>(&Pt[((4 * wave + q) * CC + li) * WPS + 8 * kb]);
            accb = mfma32(ones, b[q], accb);
        }
        // rows of X: row r of the staged tile is image row ty0 - 1 + r, and
        // with dP row q it is tap row dy + 1 = r - (4 wave + q)
#pragma unroll
        for (int x = 0; x < 6; ++x) {
            const short* row = &Xt[((4 * wave + x) * CC + li) * WXS + WX0 + 8 * kb];
            const uint4 d = *reinterpret_cast<const uint4*>(row);
            const uint32_t dl = *reinterpret_cast<const uint32_t*>(row - 2), dr = *reinterpret_cast<const uint32_t*>(row + 8);
            const uint32_t m1 = __builtin_amdgcn_alignbyte(d.y, d.x, 2), m2 = __builtin_amdgcn_alignbyte(d.z, d.y, 2),
                           m3 = __builtin_amdgcn_alignbyte(d.w, d.z, 2);
            const uint4 al = make_uint4(__builtin_amdgcn_alignbyte(d.x, dl, 2), m1, m2, m3);   // cells x - 1
            const uint4 ar = make_uint4(m1, m2, m3, __builtin_amdgcn_alignbyte(dr, d.w, 2));   // cells x + 1
            const s8 a[3] = {__builtin_bit_cast(s8, al), __builtin_bit_cast(s8, d), __builtin_bit_cast(s8, ar)};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (x - q >= 0 && x - q <= 2) {
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx) acc[3 * (x - q) + dx] = mfma32(a[dx], b[q], acc[3 * (x - q) + dx]);
                }
        }
        // the input gradients of the same rows
        if constexpr (!FIRST) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                s4 bd[9][2];
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int t = 0; t < 9; ++t)   // the cell at (1 - t / 3, 1 - t % 3) from this lane's
                        bd[t][h] = *reinterpret_cast<const s4*>(
                            &buf[((4 * wave + q + 2 - t / 3) * PW + 16 * h + li + 2 - t % 3) * CC + 4 * kb]);
                f4 ad[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                for (int t = 0; t < 9; ++t)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        ad[h] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wt[t], bd[t][h], ad[h], 0, 0, 0);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float r[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) r[i] = bf2f(xp[q][h][i]) > 0.f ? ad[h][i] : 0.f;
                    uint2 o;
                    o.x = f2bf2(r[0], r[1]);
                    o.y = f2bf2(r[2], r[3]);
                    if (cy0 + q < H4 && cx0 + 16 * h < W4)
                        *reinterpret_cast<uint2*>(dPprev + off0 + (int64_t)(q * W4 + 16 * h) * CC) = o;
                }
            }
        }
    }
    // acc[t][r] = dW[t][ci = 4 kb + r][co = li]; every row of accb is db[li]
    __syncthreads();
    static_assert(sizeof(Xt) >= 3 * kConvSums * sizeof(float), "three waves' sums");
    float* red = reinterpret_cast<float*>(Xt);
    if (wave > 0) {
        float* w = red + (wave - 1) * kConvSums;
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) w[(t * CC + 4 * kb + r) * CC + li] = acc[t][r];
        if (kb == 0) w[CONV_W + li] = accb[0];
    }
    __syncthreads();
    if (wave == 0) {
        float* out = part + (int64_t)blockIdx.x * kConvSums;
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = (t * CC + 4 * kb + r) * CC + li;
                out[i] = (acc[t][r] + red[i]) + (red[kConvSums + i] + red[2 * kConvSums + i]);
            }
        const int i = CONV_W + li;
        if (kb == 0) out[i] = (accb[0] + red[i]) + (red[kConvSums + i] + red[2 * kConvSums + i]);
    }
}

__global__ void k_fill_u32(uint32_t* p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Adam (Kingma and Ba 2015) with bias correction on fp32 master weights.
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                       int n, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Cell labels from detector keypoints: bit o of the cell holding
// (ix 2^o, iy 2^o) / 4 for every keypoint of octave o.
__global__ void k_labels(const cdvs_keypoint* __restrict__ kp, const int32_t* __restrict__ count, int kp_cap,
                         const CnnImage* __restrict__ imgs, int nimg, uint32_t* __restrict__ labels) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int img = (int)(s / kp_cap), i = (int)(s % kp_cap);
    if (img >= nimg || i >= count[img]) return;
    const cdvs_keypoint k = kp[s];
    if (k.octave < 0 || k.octave >= kMaxOctaves) return;
    const CnnImage& g = imgs[img];
    const int cx = min((k.ix << k.octave) >> 2, g.W4 - 1), cy = min((k.iy << k.octave) >> 2, g.H4 - 1);
    atomicOr(&labels[g.cell0 + (int64_t)cy * g.W4 + cx], 1u << k.octave);
}

// Active cells per (image, octave) of a mask, for the dense fallback, added to
// active[] by as many workgroups per image as its size asks for: the image's
// cell bytes are read 16 at a time from the first 16-byte boundary (the bytes
// before it and after the last whole group one at a time), and octave o's
// count of a 4-byte word is the population count of bit o of its four bytes.
// (One 1024-lane workgroup per image left 16 images' masks of 77 KB to 16
// compute units: 21 us for 16 of 1280x960 and 17 us for 128 of 640x480, now 6
// and 5 us.)
constexpr int kCountThreads = 256;
constexpr int kCountGroups = 2 * kCountThreads;   // 16-byte groups per workgroup

__device__ __forceinline__ void count_word(uint32_t x, int (&loc)[NHD]) {
#pragma unroll
    for (int o = 0; o < NHD; ++o) loc[o] += __popc(x & (0x01010101u << o));
}

__global__ __launch_bounds__(kCountThreads) void k_mask_count(const uint8_t* __restrict__ mask,
                                                             const CnnImage* __restrict__ imgs, int parts,
                                                             int32_t* __restrict__ active) {
    __shared__ int cnt[NHD];
    const int img = blockIdx.x / parts, part = blockIdx.x % parts;
    const CnnImage& g = imgs[img];
    const int64_t n = (int64_t)g.H4 * g.W4;
    const uint8_t* m = mask + g.cell0;
    const int64_t head = min(n, (int64_t)((16u - ((uint32_t)(uintptr_t)m & 15u)) & 15u));
    const int64_t ng = (n - head) / 16;   // whole 16-byte groups
    if (part > 0 && (int64_t)part * kCountGroups >= ng) return;   // uniform over the workgroup
    if (threadIdx.x < NHD) cnt[threadIdx.x] = 0;
    __syncthreads();
    int loc[NHD] = {0, 0, 0, 0, 0, 0};
    const uint4* q = reinterpret_cast<const uint4*>(m + head);
#pragma unroll
    for (int k = 0; k < kCountGroups / kCountThreads; ++k) {
        const int64_t c = (int64_t)part * kCountGroups + k * kCountThreads + threadIdx.x;
        if (c < ng) {
            const uint4 v = q[c];
            count_word(v.x, loc);
            count_word(v.y, loc);
            count_word(v.z, loc);
            count_word(v.w, loc);
        }
    }
    // the bytes before the first group and after the last
    const int64_t tail0 = head + 16 * ng, rest = head + (n - tail0);
    if (part == 0 && threadIdx.x < rest) {
        const int64_t j = threadIdx.x;
        count_word(m[j < head ? j : tail0 + (j - head)], loc);
    }
#pragma unroll
    for (int o = 0; o < NHD; ++o) {
        int v = loc[o];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if ((threadIdx.x & 63) == 0 && v) atomicAdd(&cnt[o], v);
    }
    __syncthreads();
    if (threadIdx.x < NHD && cnt[threadIdx.x]) atomicAdd(&active[img * kMaxOctaves + threadIdx.x], cnt[threadIdx.x]);
}

// All of a backward pass's sums in one launch: the head's rows, then the
// layers'.  (A launch for each takes 4.6 us, mostly its latency: one for all
// took the training step of 32 images 640x480 from 194 to 183 us, of one image
// from 78 to 68.)
constexpr int kHeadBlocks = (kHeadSums + kSumCols - 1) / kSumCols, kConvBlocks = (kConvSums + kSumCols - 1) / kSumCols;
__global__ __launch_bounds__(kSumCols * kSumRows) void k_sum_all(const float* __restrict__ rows, int head_rows,
                                                                 int conv_rows, float* __restrict__ grad,
                                                                 float* __restrict__ loss) {
    const int b = blockIdx.x;
    const float* conv = rows + (int64_t)head_rows * kHeadRow;
    if (b < kHeadBlocks) {   // uniform
        sum_parts(b, rows, head_rows, kHeadRow, kHeadSums, grad + kCnnLayers * LAYER_P, loss);
    } else {
        const int l = (b - kHeadBlocks) / kConvBlocks;
        sum_parts((b - kHeadBlocks) % kConvBlocks, conv + (int64_t)l * conv_rows * kConvSums, conv_rows, kConvSums,
                  kConvSums, grad + l * LAYER_P, nullptr);
    }
}

// Workgroups of the backward kernels that leave a row of sums each: of the
// head one per 256 cells, or wgrid of them with a longer range each; of a
// layer's weights one per tile, or wgrid with several.
int head_groups(int64_t ncells, int wgrid) {
    return (int)std::max<int64_t>(1, std::min<int64_t>((ncells + 255) / 256, wgrid));
}
int conv_groups(int ntiles, int wgrid) { return std::max(1, std::min(ntiles, wgrid)); }

}  // namespace

int64_t cnn_sum_floats(int64_t ncells, int ntiles, int wgrid) {
    return (int64_t)head_groups(ncells, wgrid) * kHeadRow + (int64_t)kCnnLayers * conv_groups(ntiles, wgrid) * kConvSums;
}

hipError_t launch_cnn_forward(const uint8_t* images, const float* params, short* frag, const CnnImage* imgs,
                              const int32_t* owner, int ntiles, short* acts, int64_t ncells, float* logits,
                              uint8_t* mask, float zthr, hipStream_t s) {
    if (ntiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cnn_pack, dim3(9), dim3(256), 0, s, params, frag);
    if (acts)
        hipLaunchKernelGGL(k_cnn_infer<true>, dim3(ntiles), dim3(FTHREADS), 0, s, images, params, frag, imgs, owner, acts,
                           ncells, logits, mask, zthr);
    else
        hipLaunchKernelGGL(k_cnn_infer<false>, dim3(ntiles), dim3(FTHREADS), 0, s, images, params, frag, imgs, owner,
                           nullptr, ncells, logits, mask, zthr);
    return hipGetLastError();
}

hipError_t launch_cnn_backward(const uint8_t* images, const float* params, const short* acts, int64_t ncells,
                               const CnnImage* imgs, int nimg, const int32_t* owner, int ntiles,
                               const float* logits, const uint32_t* labels, const float* pos_w, short* dbuf,
                               float* grad, float* loss, int wgrid, float* rows, hipStream_t s) {
    short* dA = dbuf;
    short* dB = dbuf + ncells * CC;
    const int64_t groups = (ncells + 255) / 256;
    const int hgrid = head_groups(ncells, wgrid), parts = conv_groups(ntiles, wgrid);
    const int per_block = (int)((groups + hgrid - 1) / hgrid) * 256;
    float* conv_rows = rows + (int64_t)hgrid * kHeadRow;
    hipLaunchKernelGGL(k_head_bwd, dim3(hgrid), dim3(256), 0, s, acts + (int64_t)(kCnnLayers - 1) * ncells * CC,
                       params, logits, labels, pos_w, imgs, nimg, ncells, per_block, dA, rows);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    for (int l = kCnnLayers - 1; l >= 0; --l) {
        const float* W = params + l * LAYER_P;
        const short* Xprev = l > 0 ? acts + (int64_t)(l - 1) * ncells * CC : nullptr;
        float* out = conv_rows + (int64_t)l * parts * kConvSums;
        const dim3 wg(parts);
        if (l == 0)
            hipLaunchKernelGGL(k_conv_bwd<true>, wg, dim3(256), 0, s, images, nullptr, dA, nullptr, imgs, owner, ntiles, out,
                               nullptr);
        else
            hipLaunchKernelGGL(k_conv_bwd<false>, wg, dim3(256), 0, s, images, Xprev, dA, W, imgs, owner, ntiles, out, dB);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (l > 0) {
            short* t = dA;
            dA = dB;
            dB = t;
        }
    }
    hipLaunchKernelGGL(k_sum_all, dim3(kHeadBlocks + kCnnLayers * kConvBlocks), dim3(kSumCols * kSumRows), 0, s, rows, hgrid,
                       parts, grad, loss);
    return hipGetLastError();
}

hipError_t launch_cnn_adam(float* p, const float* g, float* m, float* v, int step, float lr, float b1, float b2,
                           float eps, hipStream_t s) {
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((kCnnParams + 255) / 256), dim3(256), 0, s, p, g, m, v, kCnnParams, lr, b1, b2, eps,
                       c1, c2);
    return hipGetLastError();
}

hipError_t launch_cnn_labels(const cdvs_keypoint* kp, const int32_t* count, int kp_cap, const CnnImage* imgs, int nimg,
                             int64_t ncells, uint32_t* labels, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((ncells + 255) / 256)), dim3(256), 0, s, labels, ncells);
    const int64_t slots = (int64_t)nimg * kp_cap;
    hipLaunchKernelGGL(k_labels, dim3((unsigned)((slots + 255) / 256)), dim3(256), 0, s, kp, count, kp_cap, imgs, nimg,
                       labels);
    return hipGetLastError();
}

hipError_t launch_mask_count(const uint8_t* mask, const CnnImage* imgs, int nimg, int64_t max_cells, int32_t* active,
                             hipStream_t s) {
    const int parts = (int)std::max<int64_t>(1, (max_cells / 16 + kCountGroups - 1) / kCountGroups);
    hipLaunchKernelGGL(k_mask_count, dim3((unsigned)((int64_t)nimg * parts)), dim3(kCountThreads), 0, s, mask, imgs, parts,
                       active);
    return hipGetLastError();
}

}  // namespace cdvs
