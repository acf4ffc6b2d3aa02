// Kernels of the 3-D U-Net dose denoiser (gfx950): BF16 activations and
// weights on the matrix cores (v_mfma_f32_16x16x32_bf16) with FP32
// accumulation, channels-last tensors [n][z][y][x][c].
//
// Convolutions are 3x3x3, stride 1, zero padding 1, as implicit GEMMs:
//   forward       out[v][co]  = sum_{tap,ci} in[v+off(tap)][ci] * W[co][tap*Cin+ci]
//   data grad     din[v][ci]  = forward of dout with W'[ci][tap'*Cout+co] = W[co][(26-tap')*Cin+ci]
//   weight grad   dW[co][tap*Cin+ci] = sum_v dout[v][co] * in[v+off(tap)][ci]
// MFMA operand layout (16x16x32, verified on gfx950): lane l holds
// A[l%16][8(l/16)..+7], B[8(l/16)..+7][l%16]; the result D[4(l/16)+i][l%16].
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

namespace pmc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// an 8-byte store that may sit at any 2-byte boundary (a caller's tensor)
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));
#define GLOBAL __attribute__((address_space(1)))
#define LOCAL __attribute__((address_space(3)))

#define DEV __device__ __forceinline__

// negative slope of the leaky ReLU after every convolution
constexpr float kLeak = 0.01f;

DEV float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// round-to-nearest-even float -> bf16 bits (finite inputs)
DEV uint16_t f2bf(float f)
{
    const uint32_t u = __float_as_uint(f);
    const uint32_t r = u + 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(r >> 16);
}

// Grids: the network's [n][D][H][W] and the caller's compact [n][d][h][w]
// (d <= D, h <= H, w <= W) placed at its origin; outside it the input is
// zero (no dose, density 0) and no output is written.
struct Region {
    int D, H, W, d, h, w;
    // compact index of network voxel v, or -1 outside the caller's grid
    DEV long long compact(size_t v) const
    {
        const int x = (int)(v % W);
        size_t r = v / W;
        const int y = (int)(r % H);
        r /= H;
        const int z = (int)(r % D);
        const size_t n = r / D;
        if (x >= w || y >= h || z >= d) return -1;
        return (long long)(((n * d + z) * h + y) * w + x);
    }
};

// ------------------------------------------------------------ convolution

// Forward convolution through LDS.  A workgroup of eight waves computes a 16
// (x) x 8 (y) x 4 (z) block of output voxels (each wave 16 x 4 x 1, as four
// 16-voxel tiles) for 16*NB output channels.  The input is consumed in stages
// of QC chunks of 8 channels (one 16-byte voxel entry each): the block's halo
// (18 x 10 x 6 voxels) and the stage's weights (28 taps x 16*NB output
// channels, tap 27 the zero padding of K to 7 x 32) are copied straight from
// global memory into LDS (buffer loads to LDS; a lane past the tensor's end,
// which is where voxels outside the grid are sent, reads zero), and every
// operand is an LDS read.  K order inside a chunk: 4 taps x 8 channels per
// MFMA K-step (lane group g takes tap 4*s + g), i.e. weight column tap*Cin +
// 8*c + e.  The weights are the MFMA's A operand, so that a lane ends up with
// four consecutive output channels of one voxel and a wave stores whole rows.
// With a coarse source (Cc > 0) the input is the decoder's concatenation
// [nearest upsampling of coarse (Cc channels, half resolution), in (Cin - Cc
// channels)], read from both without forming it.
// What bounds it: the rate of L2 requests and L1 lookups, one for every piece
// of a voxel's channels a stage copies.  With one chunk a stage and 64 x 2 x 2
// blocks (4.1 halo voxels per output voxel, against 2.1 here) 96 -> 32
// channels on 80 x 64 x 64 voxels made 2.9e7 L2 requests in 115 us, 82% of one
// per channel and cycle, with the LDS 14% and the matrix cores 20% busy, and
// took 134 us; this block shape alone 89 us (1.5e7 requests), with two chunks
// a stage (32-byte pieces) 70 us.  48 -> 16 on 160 x 128 x 128: 328, 201 and
// 153 us.
// kPipe: two buffers, the copies of stage c+1 overlap the arithmetic of stage
// c; else one, and the workgroups on a CU (three with NB = 1, two with NB = 2)
// overlap each other.
// kFlat: one z plane, 64 x 8 x 1 voxels.
template <int NB, int QC, bool kFlat>
struct FwdTile {
    static constexpr int TX = kFlat ? 64 : 16, TY = 8, TZ = kFlat ? 1 : 4, WAVES = 8;
    static constexpr int HX = TX + 2, HY = TY + 2, HZ = TZ + 2;
    static constexpr int NHALO = HX * HY * HZ;                  // voxels
    static constexpr int HBLK = (NHALO * QC + 63) / 64;         // 64-entry copies of the halo
    static constexpr int WBLK = 28 * NB * QC / 4;               // and of the weights
    static constexpr int NENT = 64 * (HBLK + WBLK);
};

// What a convolution's epilogue does beside or instead of storing its output:
// what would otherwise read the whole output back.
//   kPool: also stores the 2x2x2 average of the stored (BF16) output;
//   kSplit: the output is the gradient of a concatenation [upsampled coarse
//     (Cc channels), skip]: channels below Cc are summed over the 2x2x2
//     children and stored as the coarse gradient, the others go to the skip's;
//   kHead (16 output channels): the network's head, out = dose + scale *
//     (w . d1 + b) on the caller's grid, d1 being the rounded output, which is
//     stored only if asked for.
// The sums run in the order in which a kernel of its own would take them.  At
// 160 x 128 x 128 (us, convolutions and kernels of their own against this): the
// three encoder layers with their pooling 96 and 78, the last decoder layer
// with the head 142 and 128, the three decoder gradients 386 and 248.
constexpr int kPlain = 0, kPool = 1, kSplit = 2, kHead = 3;
struct FwdAfter {
    uint16_t* half;   // kPool: pooled output; kSplit: coarse gradient
    uint16_t* rest;   // kSplit: skip gradient
    int Cc;           // kSplit: channels of the coarse gradient (a multiple of a workgroup's)
    const float *w, *b, *dose, *scale;   // kHead
    float* res;
    Region rg;
};

template <int NB, int QC, bool kPipe, int kMinWaves, int kAfter, bool kFlat>
__global__ void __launch_bounds__(512, kMinWaves)
    conv3d_fwd_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ coarse, int Cc,
                      const uint16_t* __restrict__ wt, const float* __restrict__ bias, uint16_t* __restrict__ out,
                      int N, int D, int H, int W, int Cin, int Cout, int Kp, int relu, FwdAfter after)
{
    using T = FwdTile<NB, QC, kFlat>;
    constexpr int WAVES = T::WAVES;
    // two distinct LDS objects, so that the compiler's wait for the copies
    // into one is not placed before reads of the other
    __shared__ __attribute__((aligned(16))) u32x4 buf0[T::NENT];
    __shared__ __attribute__((aligned(16))) u32x4 buf1[kPipe ? T::NENT : 4];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, g = lane >> 4;
    const int n_yb = (H + T::TY - 1) / T::TY;
    const int yb = blockIdx.y % n_yb, cg = blockIdx.y / n_yb;
    const int n_zb = (D + T::TZ - 1) / T::TZ;
    const int zb = blockIdx.z % n_zb, n = blockIdx.z / n_zb;
    const int x0 = blockIdx.x * T::TX, y0 = T::TY * yb, z0 = T::TZ * zb;
    const int co0 = cg * 16 * NB;
    const int n_chunks = Cin / 8;
    const int Cs = Cin - Cc;   // channels of `in`
    const int Hc = H >> 1, Wc = W >> 1;
    // buffer descriptors: byte offsets up to the tensors' sizes; kOutside is
    // past every tensor (all are below 2^32 - 16 bytes, checked by the host)
    constexpr uint32_t kOutside = 0xFFFFFFF0u;
    constexpr int kRaw = 0x00020000;
    const uint32_t nv = (uint32_t)((size_t)N * D * H * W);
    const auto rs_in = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(in), 0, (int)(nv * (uint32_t)Cs * 2u), kRaw);
    const auto rs_co = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(coarse), 0,
                                                         (int)((nv >> 3) * (uint32_t)Cc * 2u), kRaw);
    const auto rs_wt = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(wt), 0,
                                                         (int)((uint32_t)Cout * (uint32_t)Kp * 2u), kRaw);
    // copy the stage from chunk c on (halo, then weights) into dst: 64-entry
    // blocks dealt to the waves in turn, lane l of a block writing entry
    // 64 * blk + l.  The byte offsets of a lane's entries do not depend on the
    // chunk, which only moves the (scalar) base by 16 bytes: computed once.
    // With two chunks a stage an entry's chunk is its parity, exchanged every
    // eight voxels of a row (output channels of a tap), so that 16 neighbours
    // of one chunk lie in 16 different bank groups.
    constexpr int kBlk = T::HBLK + T::WBLK, kPer = (kBlk + WAVES - 1) / WAVES;
    uint32_t off_in[kPer], off_co[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int blk = wave + WAVES * q;
        off_in[q] = kOutside;
        off_co[q] = kOutside;
        if (blk < T::HBLK) {
            const int e = (blk * 64 + lane) / QC;
            const int hx = e % T::HX, r2 = e / T::HX;
            const int hy = r2 % T::HY, hz = r2 / T::HY;
            const int x = x0 + hx - 1, y = y0 + hy - 1, z = z0 + hz - 1;
            const uint32_t part = QC == 2 ? 16u * ((lane & 1) ^ ((hx >> 3) & 1)) : 0u;
            if (e < T::NHALO && x >= 0 && x < W && y >= 0 && y < H && z >= 0 && z < D) {
                off_in[q] = (uint32_t)(((n * D + z) * H + y) * W + x) * (uint32_t)Cs * 2u + part;
                if (Cc)
                    off_co[q] = (uint32_t)(((n * (D >> 1) + (z >> 1)) * Hc + (y >> 1)) * Wc + (x >> 1)) * (uint32_t)Cc * 2u + part;
            }
        } else {
            const int qq = ((blk - T::HBLK) * 64 + lane) / QC, tap = qq / (16 * NB), co = co0 + qq % (16 * NB);
            const uint32_t part = QC == 2 ? 16u * ((lane & 1) ^ ((qq >> 3) & 1)) : 0u;
            if (tap < 27 && co < Cout) off_in[q] = (uint32_t)(co * Kp + tap * Cin) * 2u + part;
        }
    }
    auto issue = [&](int c, u32x4* dst) __attribute__((always_inline)) {
        const bool from_coarse = 8 * c < Cc;
        const int s_in = from_coarse ? 16 * c : 16 * c - 2 * Cc;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int blk = wave + WAVES * q;
            LOCAL void* to = (LOCAL void*)(dst + blk * 64);
            if (blk < T::HBLK) {
                if (from_coarse)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_co, to, 16, (int)off_co[q], s_in, 0, 0);
                else
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_in, to, 16, (int)off_in[q], s_in, 0, 0);
            } else if (kBlk % WAVES == 0 || blk < kBlk) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_wt, to, 16, (int)off_in[q], 16 * c, 0, 0);
            }
        }
    };
    f32x4 acc[4][NB];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[t][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // this wave's voxels: x0 + xw + m, y0 + yw + t, z0 + zw; its lane's first halo
    // entry and first weight entry
    const int xw = kFlat ? 16 * (wave >> 1) : 0, yw = 4 * (wave & 1), zw = kFlat ? 0 : wave >> 1;
    const int vox0 = (zw * T::HY + yw) * T::HX + xw + m;
    const int wt0 = g * 16 * NB + m;
    auto compute = [&](const u32x4* bf, int q) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 7; ++s) {
            const int tap = 4 * s + g;
            const int kz = tap / 9, ky = (tap / 3) % 3, kx = tap % 3;
            // (for the padding tap the index stays inside the buffer; the
            // entry read is discarded)
            const int v = QC * (vox0 + (kz * T::HY + ky) * T::HX + kx) + (QC == 2 ? q ^ (((m + kx) >> 3) & 1) : 0);
            const int w0 = 64 * T::HBLK + QC * wt0 + (QC == 2 ? q ^ ((m >> 3) & 1) : 0);
            bf16x8 a[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) a[j] = __builtin_bit_cast(bf16x8, bf[w0 + QC * (64 * NB * s + 16 * j)]);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const u32x4 e = bf[v + QC * T::HX * t];
                const bf16x8 b = s < 6 || tap < 27 ? __builtin_bit_cast(bf16x8, e) : (bf16x8){};
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j], b, acc[t][j], 0, 0, 0);
            }
        }
    };
    auto stage = [&](const u32x4* bf) __attribute__((always_inline)) {
        compute(bf, 0);
        if constexpr (QC == 2) compute(bf, 1);
    };
    // vmcnt(0), other counters untouched: this wave's copies have landed
    constexpr int kWaitCopies = 0x0F70;
    if constexpr (kPipe) {
        issue(0, buf0);
        for (int c = 0; c < n_chunks; c += 2 * QC) {
            __builtin_amdgcn_s_waitcnt(kWaitCopies);
            __syncthreads();   // the stage in buf0 complete; buf1 no longer read
            if (c + QC < n_chunks) issue(c + QC, buf1);
            stage(buf0);
            if (c + QC >= n_chunks) break;
            __builtin_amdgcn_s_waitcnt(kWaitCopies);
            __syncthreads();   // the stage in buf1 complete; buf0 no longer read
            if (c + 2 * QC < n_chunks) issue(c + 2 * QC, buf0);
            stage(buf1);
        }
    } else {
        for (int c = 0; c < n_chunks; c += QC) {
            if (c) __syncthreads();   // buf0 no longer read
            issue(c, buf0);
            __builtin_amdgcn_s_waitcnt(kWaitCopies);
            __syncthreads();
            stage(buf0);
        }
    }
    // lane (m, g) holds output channels co0 + 16 j + 4 g .. + 3 of voxel m
    const int x = x0 + xw + m, z = z0 + zw;
    const bool in_xz = x < W && z < D;
    // the block's channels go to a coarse gradient (kSplit): nothing to store per voxel
    const bool to_half = kAfter == kSplit && co0 < after.Cc;
    u32x2 o[4][NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int co = co0 + 16 * j + 4 * g;
        float bv[4] = {0.f, 0.f, 0.f, 0.f};
        if (bias && co < Cout)   // (Cout is a multiple of 8)
#pragma unroll
            for (int i = 0; i < 4; ++i) bv[i] = bias[co + i];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int y = y0 + yw + t;
            uint32_t q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float v = acc[t][j][i] + bv[i];
                if (relu) v = v > 0.f ? v : kLeak * v;
                q[i] = f2bf(v);
            }
            o[t][j] = (u32x2){q[0] | (q[1] << 16), q[2] | (q[3] << 16)};
            if (!in_xz || y >= H || co >= Cout) continue;
            const size_t vox = (((size_t)n * D + z) * H + y) * W + x;
            if constexpr (kAfter == kSplit) {
                if (!to_half)
                    *reinterpret_cast<u32x2_any*>(after.rest + vox * (Cout - after.Cc) + (co - after.Cc)) = o[t][j];
            } else if (kAfter != kHead || out) {
                *reinterpret_cast<u32x2_any*>(out + vox * Cout + co) = o[t][j];
            }
        }
    }
    if constexpr (kAfter == kPool || kAfter == kSplit) {
        if (kAfter == kSplit && !to_half) return;   // (the whole workgroup)
        // sums over 2x2x2 voxels in the order z, y, x: the wave of the even
        // plane leaves its four-voxel sums in LDS, that of the odd plane adds
        // its own; even lanes hold the x pairs
        f32x4* const xch = reinterpret_cast<f32x4*>(buf0);
        static_assert(8 * NB * 64 <= T::NENT, "the four-voxel sums fit a stage's buffer");
        auto quad = [&](int tp, int j, f32x4 s) {
#pragma unroll
            for (int dy = 0; dy < 2; ++dy) {
                const u32x2 own = o[2 * tp + dy][j];
                const u32x2 next = {(uint32_t)__shfl_xor((int)own.x, 1), (uint32_t)__shfl_xor((int)own.y, 1)};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    s[i] += __uint_as_float(i & 1 ? own[i >> 1] & 0xFFFF0000u : own[i >> 1] << 16);
                    s[i] += __uint_as_float(i & 1 ? next[i >> 1] & 0xFFFF0000u : next[i >> 1] << 16);
                }
            }
            return s;
        };
        auto slot = [&](int tp, int j) { return ((((wave >> 2) * 2 + (wave & 1)) * 2 + tp) * NB + j) * 64 + lane; };
        __syncthreads();   // the stage's buffer is no longer read
        if (!(zw & 1)) {
#pragma unroll
            for (int tp = 0; tp < 2; ++tp)
#pragma unroll
                for (int j = 0; j < NB; ++j) xch[slot(tp, j)] = quad(tp, j, (f32x4){0.f, 0.f, 0.f, 0.f});
        }
        __syncthreads();
        if (zw & 1) {
            const int Ch = kAfter == kSplit ? after.Cc : Cout;
#pragma unroll
            for (int tp = 0; tp < 2; ++tp)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const f32x4 s = quad(tp, j, xch[slot(tp, j)]);
                    const float k = kAfter == kPool ? 0.125f : 1.f;
                    const int co = co0 + 16 * j + 4 * g, y = y0 + yw + 2 * tp;
                    if (!in_xz || (m & 1) || y >= H || co >= Ch) continue;
                    const size_t vox = (((size_t)n * (D >> 1) + (z >> 1)) * Hc + (y >> 1)) * Wc + (x >> 1);
                    *reinterpret_cast<u32x2*>(after.half + vox * Ch + co) =
                        (u32x2){(uint32_t)f2bf(k * s[0]) | ((uint32_t)f2bf(k * s[1]) << 16),
                                (uint32_t)f2bf(k * s[2]) | ((uint32_t)f2bf(k * s[3]) << 16)};
                }
        }
    }
    if constexpr (kAfter == kHead) {
        // the sum over the 16 channels passes through the four lane groups in
        // turn; group g then writes row g
        float hw[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) hw[i] = after.w[4 * g + i];
        const float sc = fmaxf(after.scale[0], 1e-30f);
        float s[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            s[t] = after.b[0];
#pragma unroll
            for (int gg = 0; gg < 4; ++gg) {
                float v = s[t];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    v += hw[i] * __uint_as_float(i & 1 ? o[t][0][i >> 1] & 0xFFFF0000u : o[t][0][i >> 1] << 16);
                s[t] = __shfl(v, 16 * gg + m);
            }
        }
        const float sg = g == 0 ? s[0] : (g == 1 ? s[1] : (g == 2 ? s[2] : s[3]));
        const int y = y0 + yw + g;
        if (x < after.rg.w && y < after.rg.h && z < after.rg.d) {
            const size_t vc = (((size_t)n * after.rg.d + z) * after.rg.h + y) * after.rg.w + x;
            after.res[vc] = after.dose[vc] + sc * sg;
        }
    }
}

// W'[ci][tap'*Cout + co] = W[co][(26 - tap')*Cin + ci]  (row length Kp'); one
// launch flips the layers of a whole backward pass (grid y: layer), where a
// launch of its own took 4.7 us for each of six
struct FlipLayer {
    const uint16_t* w;
    uint16_t* wf;
    int Cin, Cout, Kp, Kpf;
};
struct FlipLayers {
    FlipLayer l[7];
};
__global__ void flip_weights_kernel(FlipLayers f)
{
    const FlipLayer& a = f.l[blockIdx.y];
    const int total = a.Cin * a.Kpf;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
        const int ci = i / a.Kpf, kk = i - ci * a.Kpf;
        uint16_t v = 0;
        if (kk < 27 * a.Cout) {
            const int tp = kk / a.Cout, co = kk - tp * a.Cout;
            v = a.w[(size_t)co * a.Kp + (26 - tp) * a.Cin + ci];
        }
        a.wf[i] = v;
    }
}

// Weight gradient: dW[co][tap][ci] += sum over input voxels v' of in[v'][ci]
// dout[v' - off(tap)][co], off(tap) = (kz, ky, kx) - 1.  The voxels are the K
// dimension of the product, so both operands have voxels along K while the
// tensors are channels-last: they are copied to LDS as they are and read with
// the transposing LDS load (ds_read_b64_tr_b16: four voxels of one channel per
// lane), no shifted or transposed copies.
// A workgroup of 12 waves owns a column of 32 (x) x TY (y) input voxels, 16 NCI
// input and 16 NCO output channels, and walks a run of z planes.  Per plane it
// holds the input plane (x halo of one, two buffers) and the output gradient of
// planes z-1, z, z+1 (y halo of one, a ring of four), the next plane's copies
// in flight.  A wave has one 16-channel input tile, one 16-channel output tile
// and two of the rows, and all 27 taps in 108 accumulator registers: per plane
// 6 input and 12 output-gradient fragments (each 32 voxels of a row) feed 54
// MFMAs.  Planes and rows are split by the input's, x by the output's, so that
// the smaller tensor carries the y and z halo; what lies outside the grid is
// copied as zeros.  With a coarse source (Cc > 0, a multiple of 16) the input
// is the decoder's concatenation [nearest upsampling of coarse, in], read from
// both.  At the end the waves' row slices are added in LDS and the
// workgroup adds its sums to dw, one atomic per weight.
// What bounds it: with 16 output channels the MFMA rate (48 -> 16 channels on
// 160 x 128 x 128: 113 us, 0.96 PFLOP/s; a kernel that transposed both operands
// through registers into shifted LDS copies, 2,048 workgroups in flight, was
// latency-bound at 701 us); the deeper, smaller layers the 16-20 us of the
// first copies and the final sums, which every workgroup pays once (192 -> 64
// on 40 x 32 x 32: 59 us, before 243; 64 -> 128 on 20 x 16 x 16: 31, before
// 124).
// kWide: z planes whose byte offsets do not fit the buffer loads' 32 bits: the
// copies take 64-bit addresses, lanes outside the grid those of a page of zeros.
constexpr int kWgWaves = 12;
__device__ const u32x4 kZeros[1] = {};

// 64 lanes x 16 bytes at the lanes' byte offsets of a buffer to LDS address
// `to` + 16 * lane; lanes past the buffer's end write zeros.  As an
// instruction the compiler does not see as a load, so that it does not wait
// for the copy before unrelated LDS reads: the caller waits for vmcnt(0)
// before the barrier that hands the data over.  m0 is left as it was (the
// compiler takes it for its own register and may count on its value); the wait
// states are for m0 and, should the descriptor have come from vector registers
// just before, for it.
DEV void copy_to_lds(i32x4 rsrc, uint32_t off, uint32_t to)
{
    uint32_t m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 4\n\tbuffer_load_dwordx4 %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
                 : "=&s"(m0)
                 : "s"(to), "v"(off), "s"(rsrc)
                 : "memory");
}
template <int NCI, int NCO>
struct WgTile {
    static constexpr int KS = kWgWaves / (NCI * NCO), TY = 2 * KS;
    static constexpr int IBLK = (TY * 68 + 63) / 64;            // 64-entry copies of one input tile's plane
    static constexpr int NIN = NCI * IBLK, NDO = NCO * (TY + 2);
    static constexpr int PER = (NIN + NDO + kWgWaves - 1) / kWgWaves;
};

template <int NCI, int NCO, bool kWide>
__global__ void __launch_bounds__(64 * kWgWaves, 3)
    conv3d_wgrad_kernel(const uint16_t* __restrict__ in, const uint16_t* __restrict__ coarse, int Cc,
                        const uint16_t* __restrict__ dout, float* __restrict__ dw, int D, int H, int W, int Cin, int Cout, int Kp, int n_xt, int n_yt, unsigned long long n_planes,
                        int per_block)
{
    using T = WgTile<NCI, NCO>;
    constexpr int KS = T::KS, TY = T::TY;
    // two input planes, then a ring of four output-gradient planes
    constexpr int kInBytes = 1024 * T::NIN, kDoBytes = 1024 * T::NDO;
    __shared__ __attribute__((aligned(16))) char lds[2 * kInBytes + 4 * kDoBytes];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, g = lane >> 4;
    // workgroup -> channel blocks and its run of the block's planes: plane
    // index = ((volume * n_yt + y tile) * n_xt + x tile) * D + z
    const int n_cib = (Cin + 16 * NCI - 1) / (16 * NCI);
    const int blk2 = blockIdx.x / per_block, part = blockIdx.x % per_block;
    const int ci0 = 16 * NCI * (blk2 % n_cib), co0 = 16 * NCO * (blk2 / n_cib);
    unsigned long long p = n_planes * part / per_block;
    const unsigned long long p_end = n_planes * (part + 1) / per_block;
    const size_t plane = (size_t)H * W;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(LOCAL char*)lds;
    // this wave's tiles and rows
    const int tj = wave % NCI, tc = (wave / NCI) % NCO, ks = wave / (NCI * NCO);
    // fragment reads: lane (g, m) addresses voxel 4 g + m / 4 of a row, four
    // channels from 4 (m % 4); the second half of a fragment lies 16 voxels on
    // (both operands alike, so the order along K does not matter)
    const int lane_at = (4 * g + (m >> 2)) * 32 + 8 * (m & 3);
    const int in_at = tj * T::IBLK * 1024 + 2 * ks * 34 * 32 + lane_at;
    const int do_at = tc * (TY + 2) * 1024 + 2 * ks * 32 * 32 + lane_at;
    auto frag = [&](const char* p) __attribute__((always_inline)) {
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LOCAL i16x4*)p);
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LOCAL i16x4*)(p + 512));
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    f32x4 acc[27];
#pragma unroll
    for (int t = 0; t < 27; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    while (p < p_end) {
    // the planes of one column: z_begin .. z_end - 1 of volume n
    const unsigned long long col = p / (unsigned)D;
    const int z_begin = (int)(p - col * (unsigned)D);
    const int z_end = (int)min((unsigned long long)D, z_begin + (p_end - p));
    p += z_end - z_begin;
    const int xt = (int)(col % (unsigned)n_xt), yt = (int)(col / (unsigned)n_xt % (unsigned)n_yt);
    const size_t n = (size_t)(col / (unsigned)n_xt / (unsigned)n_yt);
    const int x0 = 32 * xt, y0 = TY * yt;
    // byte offsets, within a z plane, of the entries this lane copies: blocks
    // of 64 dealt to the waves in turn, the input's tiles first
    using Offset = std::conditional_t<kWide, size_t, uint32_t>;
    constexpr Offset kOutside = kWide ? ~(Offset)0 : (Offset)0xFFFFFFF0u;
    Offset off[T::PER];
#pragma unroll
    for (int q = 0; q < T::PER; ++q) {
        const int blk = wave + kWgWaves * q;
        off[q] = kOutside;
        if (blk < T::NIN) {
            const int e = (blk % T::IBLK) * 64 + lane;
            const int row = e / 68, r2 = e % 68;
            const int x = x0 + (r2 >> 1) - 1, y = y0 + row, c = ci0 + 16 * (blk / T::IBLK) + 8 * (r2 & 1);
            if (row < TY && x >= 0 && x < W && y < H && c < Cin)
                off[q] = c < Cc ? (((Offset)(y >> 1) * (W >> 1) + (x >> 1)) * Cc + c) * 2u
                                : (((Offset)y * W + x) * (Cin - Cc) + (c - Cc)) * 2u;
        } else if (blk < T::NIN + T::NDO) {
            const int d = blk - T::NIN;
            const int x = x0 + (lane >> 1), y = y0 + d % (TY + 2) - 1, c = co0 + 16 * (d / (TY + 2)) + 8 * (lane & 1);
            if (x < W && y >= 0 && y < H && c < Cout) off[q] = (((Offset)y * W + x) * Cout + c) * 2u;
        }
    }
    // z plane -> buffer descriptor (empty outside the grid: every lane reads
    // zero); wide: its address (NULL outside)
    auto plane_at = [&](const uint16_t* t, int z, int planes, size_t bytes) {
        const bool ok = z >= 0 && z < planes;
        const uint64_t at = (uint64_t)(uintptr_t)t + (n * planes + (ok ? z : 0)) * bytes;
        if constexpr (kWide) return ok ? at : (uint64_t)0;
        else return (i32x4){(int)(uint32_t)at, (int)(uint32_t)(at >> 32), ok ? (int)(uint32_t)bytes : 0, 0x00020000};
    };
    auto copy = [&](auto from, Offset o, uint32_t to) __attribute__((always_inline)) {
        if constexpr (kWide) {
            const GLOBAL char* src = from != 0 && o != kOutside ? (const GLOBAL char*)(uintptr_t)(from + o)
                                                                : (const GLOBAL char*)&kZeros[0];
            __builtin_amdgcn_global_load_lds((const GLOBAL void*)src, (LOCAL void*)(uintptr_t)to, 16, 0, 0);
        } else {
            copy_to_lds(from, o, to);
        }
    };
    // input plane z (its own buffer) and output-gradient plane zd to LDS
    auto load = [&](int z, bool with_in, int zd) __attribute__((always_inline)) {
        const auto ri = plane_at(in, z, D, plane * (Cin - Cc) * 2), rd = plane_at(dout, zd, D, plane * Cout * 2);
        const auto rc = plane_at(coarse, z >> 1, D >> 1, (plane >> 2) * Cc * 2);
        const uint32_t ti = lds0 + (z & 1) * kInBytes, td = lds0 + 2 * kInBytes + (zd & 3) * kDoBytes;
#pragma unroll
        for (int q = 0; q < T::PER; ++q) {
            const int blk = wave + kWgWaves * q;
            if (blk < T::NIN) {
                if (with_in) copy(ci0 + 16 * (blk / T::IBLK) < Cc ? rc : ri, off[q], ti + 1024 * blk);
            } else if (blk < T::NIN + T::NDO) {
                copy(rd, off[q], td + 1024 * (blk - T::NIN));
            }
        }
    };
    // input plane z against the output gradient's planes z+1, z, z-1 (kz = 0,
    // 1, 2); at the grid's faces the products with the rows and planes outside
    // are left out (an infinite input times their zeros would not vanish)
    auto step = [&](int z) __attribute__((always_inline)) {
        const char* pin = lds + (z & 1) * kInBytes + in_at;
        const char* pd[3];
#pragma unroll
        for (int kz = 0; kz < 3; ++kz) pd[kz] = lds + 2 * kInBytes + ((z + 1 - kz) & 3) * kDoBytes + do_at;
        bf16x8 bv[2][3];
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) bv[r][kx] = frag(pin + (r * 34 + kx) * 32);
        // row 2 ks + a - 1 of the output gradient: tap ky = r + 2 - a of input row r
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const bf16x8 av[3] = {frag(pd[0] + a * 1024), frag(pd[1] + a * 1024), frag(pd[2] + a * 1024)};
            const int y = y0 + 2 * ks + a - 1;
            if (y < 0 || y >= H) continue;
#pragma unroll
            for (int kz = 0; kz < 3; ++kz) {
                if (kz != 1 && (z + 1 - kz < 0 || z + 1 - kz >= D)) continue;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int ky = r + 2 - a;
                    if (ky < 0 || ky > 2) continue;
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx) {
                        f32x4& t = acc[(kz * 3 + ky) * 3 + kx];
                        t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[kz], bv[r][kx], t, 0, 0, 0);
                    }
                }
            }
        }
    };
    constexpr int kWaitCopies = 0x0F70;   // vmcnt(0), other counters untouched
    load(z_begin, true, z_begin - 1);
    load(z_begin, false, z_begin);
    load(z_begin, false, z_begin + 1);
    __builtin_amdgcn_s_waitcnt(kWaitCopies);
    __syncthreads();
    for (int z = z_begin; z < z_end; ++z) {
        // the next plane's copies go where nothing is read during this one
        if (z + 1 < z_end) load(z + 1, true, z + 2);
        step(z);
        __builtin_amdgcn_s_waitcnt(kWaitCopies);
        __syncthreads();
    }
    }   // columns
    // add up the row slices, three taps at a time: every wave leaves its tiles
    // in the copies' LDS (no longer read; lane (g, m) holds output channels
    // 4 g .. + 3 of input channel m), then each weight's KS values are summed
    constexpr int kTiles = 3 * NCI * NCO;
    static_assert(KS * kTiles * 1024 <= (int)sizeof(lds), "the waves' tiles fit the copies' LDS");
    float* const red = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int k3 = 0; k3 < 9; ++k3) {
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                red[((ks * 3 + kx) * NCO * NCI + tc * NCI + tj) * 256 + (4 * g + i) * 16 + m] = acc[3 * k3 + kx][i];
        __syncthreads();
        for (int e = threadIdx.x; e < kTiles * 256; e += 64 * kWgWaves) {
            const int t = e >> 8, j = t % NCI, c = (t / NCI) % NCO, kx = t / (NCI * NCO);
            const int co = co0 + 16 * c + ((e >> 4) & 15), ci = ci0 + 16 * j + (e & 15);
            float v = 0.f;
#pragma unroll
            for (int q = 0; q < KS; ++q) v += red[q * kTiles * 256 + e];
            if (co < Cout && ci < Cin && v != 0.f) atomicAdd(&dw[(size_t)co * Kp + (3 * k3 + kx) * Cin + ci], v);
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------ elementwise

// Leaky-ReLU backward through the stored output (which has the sign of the
// pre-activation): the gradient of one BF16 value, rounded to BF16
DEV uint32_t relu_grad(uint32_t d, bool positive) { return positive ? d : (uint32_t)f2bf(kLeak * bf2f((uint16_t)d)); }

// the block's per-lane sums of 8 channels (channel group threadIdx.x % G) to
// the bias gradient, one atomic per block and channel
DEV void add_bias_grad(const float* acc, int G, int C, float* __restrict__ db)
{
    __shared__ float part[256 * 8];
#pragma unroll
    for (int k = 0; k < 8; ++k) part[threadIdx.x * 8 + k] = acc[k];
    __syncthreads();
    const int lanes_per_g = 256 / G;
    for (int c = threadIdx.x; c < C; c += 256) {
        float t = 0.f;
        for (int s = 0; s < lanes_per_g; ++s) t += part[(s * G + c / 8) * 8 + c % 8];
        atomicAdd(&db[c], t);
    }
}

// Gradient at a layer's pre-activation and its bias gradient in one pass over
// rows of voxels: dy[v][c] = relu'(y[v][c]) * g with g = src[v][c], or with
// kPool (the gradient of a pooled output beside that of a skip connection) g =
// src[v][c] + dpool[parent(v)][c] / 8; both roundings of g and of the product
// to BF16, db[c] += sum_v dy[v][c] of the rounded values.  src may be dy
// itself.  A lane takes 8 channels (16 bytes) of a voxel, C / 8 a power of two
// up to 32.  HBM-bound (160 x 128 x 128 x 16, with pooling: 262 MB, two
// kernels 78 us, one 47); few workgroups where the tensor is small, as
// each adds to the same C addresses.
template <bool kPool>
__global__ void __launch_bounds__(256) grad_relu_kernel(const uint16_t* src, const uint16_t* __restrict__ dpool,
                                                        const uint16_t* __restrict__ y, uint16_t* dy,
                                                        float* __restrict__ db, unsigned rows, int D, int H, int W, int C)
{
    const int G = C / 8, lg = __builtin_ctz(G);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // two rows at a time: six (four) 16-byte loads in flight per lane
    for (unsigned r0 = blockIdx.x; r0 < rows; r0 += 2 * gridDim.x) {
        const bool two = r0 + gridDim.x < rows;
        size_t base[2];
        const uint16_t* prow[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const unsigned r = k && two ? r0 + gridDim.x : r0;
            base[k] = (size_t)r * W * C;
            const unsigned t = r / (unsigned)H, yy = r - t * (unsigned)H, n = t / (unsigned)D, z = t - n * (unsigned)D;
            prow[k] = dpool + (((size_t)n * (D >> 1) + (z >> 1)) * (H >> 1) + (yy >> 1)) * (W >> 1) * C;
        }
        for (int i = threadIdx.x; i < W * G; i += 256) {
            uint4 sv[2], yv[2], pv[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                sv[k] = *reinterpret_cast<const uint4*>(src + base[k] + 8 * (size_t)i);
                yv[k] = *reinterpret_cast<const uint4*>(y + base[k] + 8 * (size_t)i);
                if (kPool)
                    pv[k] = *reinterpret_cast<const uint4*>(prow[k] + 8 * ((size_t)(i >> (lg + 1)) * G + (i & (G - 1))));
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                if (k && !two) break;
                const uint32_t sw[4] = {sv[k].x, sv[k].y, sv[k].z, sv[k].w}, yw[4] = {yv[k].x, yv[k].y, yv[k].z, yv[k].w},
                               pw[4] = {pv[k].x, pv[k].y, pv[k].z, pv[k].w};
                uint32_t o[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    o[q] = 0;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        uint32_t d = (sw[q] >> (16 * h)) & 0xFFFFu;
                        if (kPool) {
                            float v = 0.125f * bf2f((uint16_t)(pw[q] >> (16 * h)));
                            v += bf2f((uint16_t)d);
                            d = f2bf(v);
                        }
                        d = relu_grad(d, bf2f((uint16_t)(yw[q] >> (16 * h))) > 0.f);
                        acc[2 * q + h] += bf2f((uint16_t)d);
                        o[q] |= d << (16 * h);
                    }
                }
                *reinterpret_cast<uint4*>(dy + base[k] + 8 * (size_t)i) = make_uint4(o[0], o[1], o[2], o[3]);
            }
        }
    }
    add_bias_grad(acc, G, C, db);
}

// Workgroups of the reductions below; each leaves its value in an array that
// the next kernel (or the host) adds up, since atomics of all workgroups on
// one address serialise at about 12 ns each (counting the dose region with
// 1,024 of them took 15.7 us, the gradient norm's 16.5 us).
constexpr int kParts = 256;

// f(a[i]) over the grid's share of a, eight loads in flight per lane
template <class F>
DEV void each_of(size_t n, const float* __restrict__ a, F f)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    for (; i + 7 * stride < n; i += 8 * stride) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = a[i + k * stride];
#pragma unroll
        for (int k = 0; k < 8; ++k) f(v[k]);
    }
    for (; i < n; i += stride) f(a[i]);
}

// parts[b] = max of workgroup b's voxels of a (non-negative input), 0 for none
__global__ void __launch_bounds__(256) max_kernel(const float* __restrict__ a, size_t n, float* __restrict__ parts)
{
    __shared__ float part[4];
    float m = 0.f;
    each_of(n, a, [&](float v) { m = fmaxf(m, v); });
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) parts[blockIdx.x] = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
}

// network input: x[v] = (dose[v] * inv_scale, density[v] * 0.5, 0 x 6), zero
// outside the caller's grid; scale[0] = the maximum dose, from the n_parts <= 256
// shares after it, which every workgroup reads again (one kernel for the maximum
// with an atomic per workgroup, behind a clear of its target, took 16.5 us on
// 160 x 128 x 128 voxels where the shares take 7).  Bound by its bytes: 24 per
// voxel, 13 us.
__global__ void __launch_bounds__(256) make_input_kernel(const float* __restrict__ dose, const float* __restrict__ rho,
                                                         float* __restrict__ scale, int n_parts,
                                                         uint4* __restrict__ x, size_t nvox, Region rg)
{
    __shared__ float part[4];
    float m = (int)threadIdx.x < n_parts ? scale[1 + threadIdx.x] : 0.f;
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    m = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
    if (blockIdx.x == 0 && threadIdx.x == 0) scale[0] = m;
    const float inv = 1.0f / fmaxf(m, 1e-30f);
    for (size_t v = blockIdx.x * (size_t)blockDim.x + threadIdx.x; v < nvox; v += (size_t)gridDim.x * blockDim.x) {
        const long long vc = rg.compact(v);
        const uint32_t both = vc >= 0 ? (uint32_t)f2bf(dose[vc] * inv) | (uint32_t)f2bf(rho[vc] * 0.5f) << 16 : 0u;
        x[v] = make_uint4(both, 0u, 0u, 0u);
    }
}

// part[b] = workgroup b's number of voxels with dose >= frac * scale (the dose
// region that normalises the loss)
__global__ void __launch_bounds__(256) region_count_kernel(const float* __restrict__ dose, size_t n,
                                                           const float* __restrict__ scale, float frac,
                                                           unsigned int* __restrict__ parts)
{
    __shared__ unsigned int part[4];
    const float thr = frac * scale[0];
    unsigned int c = 0;
    each_of(n, dose, [&](float a) { c += a >= thr; });
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) parts[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// Squared error in normalised units over the dose region,
// L = sum_v ((out_v - t_v) / scale)^2 / n_region (every voxel contributes;
// n_region, the count of voxels with dose >= 1% of scale, sets the scale of
// the gradients), the head backward: g_v = dL/d(head pre-activation) =
// 2 (out_v - t_v) / scale / n_region, dw[c] += sum_v g_v d1[v][c], db += sum_v
// g_v; and the backward of the last layer's leaky ReLU, whose output d1 is at
// hand: dd1[v][c] = relu'(d1[v][c]) * bf16(g_v w[c]), dbias[c] += sum_v
// dd1[v][c].  loss_part[b] = workgroup b's share of L (host memory).  C = 16
// channels: one 32-byte row per voxel.  Block partial sums meet in LDS; one
// atomic per block and quantity.  HBM-bound (160 x 128 x 128: 190 MB, 42
// us; 83 us as two kernels).
__global__ void __launch_bounds__(256) loss_head_bwd_kernel(const float* __restrict__ out,
                                                            const float* __restrict__ target,
                                                            const float* __restrict__ scale,
                                                            const uint16_t* __restrict__ d1,
                                                            const float* __restrict__ w,
                                                            uint16_t* __restrict__ dd1, float* __restrict__ dw,
                                                            float* __restrict__ db, float* __restrict__ dbias,
                                                            double* __restrict__ loss_part, size_t nvox,
                                                            const unsigned int* __restrict__ region_part, int n_part)
{
    __shared__ float sg[4][33];
    __shared__ double sl[4];
    __shared__ unsigned int sr[4];
    const int wave = threadIdx.x >> 6;
    unsigned int n_region = (int)threadIdx.x < n_part ? region_part[threadIdx.x] : 0u;
    for (int o = 32; o > 0; o >>= 1) n_region += __shfl_xor(n_region, o);
    if ((threadIdx.x & 63) == 0) sr[wave] = n_region;
    __syncthreads();
    const float inv_count = 1.0f / (float)max(1u, sr[0] + sr[1] + sr[2] + sr[3]);
    const float sc = fmaxf(scale[0], 1e-30f);
    const float isc = 1.0f / sc;
    float wv[16], sums[33];   // gradients of w, then b, then the bias
#pragma unroll
    for (int c = 0; c < 16; ++c) wv[c] = w[c];
#pragma unroll
    for (int c = 0; c < 33; ++c) sums[c] = 0.f;
    double l = 0.0;
    // two voxels at a time: eight loads in flight per lane
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t v0 = blockIdx.x * (size_t)blockDim.x + threadIdx.x; v0 < nvox; v0 += 2 * stride) {
        const bool two = v0 + stride < nvox;
        float ov[2], tv[2];
        uint4 src[2][2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const size_t v = k && two ? v0 + stride : v0;
            ov[k] = out[v];
            tv[k] = target[v];
#pragma unroll
            for (int h = 0; h < 2; ++h) src[k][h] = reinterpret_cast<const uint4*>(d1 + v * 16)[h];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (k && !two) break;
            const float e = (ov[k] - tv[k]) * isc;
            l += (double)e * e;
            const float g = 2.f * e * inv_count;
            sums[16] += g;
            uint4* dst = reinterpret_cast<uint4*>(dd1 + (v0 + k * stride) * 16);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint4 q = src[k][h];
                const uint32_t in[4] = {q.x, q.y, q.z, q.w};
                uint32_t o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int c = 8 * h + 2 * i;
                    const float lo = __uint_as_float(in[i] << 16), hi = __uint_as_float(in[i] & 0xFFFF0000u);
                    sums[c] += g * lo;
                    sums[c + 1] += g * hi;
                    const uint32_t dlo = relu_grad(f2bf(g * wv[c]), lo > 0.f), dhi = relu_grad(f2bf(g * wv[c + 1]), hi > 0.f);
                    sums[17 + c] += bf2f((uint16_t)dlo);
                    sums[18 + c] += bf2f((uint16_t)dhi);
                    o[i] = dlo | (dhi << 16);
                }
                dst[h] = make_uint4(o[0], o[1], o[2], o[3]);
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        l += __shfl_xor(l, o);
#pragma unroll
        for (int c = 0; c < 33; ++c) sums[c] += __shfl_xor(sums[c], o);
    }
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int c = 0; c < 33; ++c) sg[wave][c] = sums[c];
        sl[wave] = l;
    }
    __syncthreads();
    const int c = threadIdx.x;
    if (c < 33) {
        const float t = sg[0][c] + sg[1][c] + sg[2][c] + sg[3][c];
        atomicAdd(c < 16 ? &dw[c] : (c == 16 ? db : &dbias[c - 17]), t);
    } else if (c == 64) {
        loss_part[blockIdx.x] = (sl[0] + sl[1] + sl[2] + sl[3]) * inv_count;
    }
}

// Adam on FP32 master parameters; refreshes the BF16 copies of the
// convolution weights (p_bf == NULL for parameters kept in FP32)
// part[b] = workgroup b's share of the sum of squares of a float vector, in
// FP64 (host memory)
__global__ void __launch_bounds__(256) sqnorm_kernel(const float* __restrict__ g, size_t n, double* __restrict__ parts)
{
    __shared__ double part[4];
    double acc = 0.0;
    each_of(n, g, [&](float v) { acc += (double)v * (double)v; });
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) parts[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// Adam on gradient gs * g (gs: the caller's clipping factor, 1 = plain)
__global__ void adam_kernel(float* __restrict__ p, float* __restrict__ g, float* __restrict__ m1,
                            float* __restrict__ m2, uint16_t* __restrict__ p_bf, size_t n, float lr,
                            float b1, float b2, float eps, float c1, float c2, float gs)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const float gi = gs * g[i];
        const float a = b1 * m1[i] + (1.f - b1) * gi;
        const float s = b2 * m2[i] + (1.f - b2) * gi * gi;
        m1[i] = a;
        m2[i] = s;
        const float v = p[i] - lr * (a / c1) / (sqrtf(s / c2) + eps);
        p[i] = v;
        g[i] = 0.f;
        if (p_bf) p_bf[i] = f2bf(v);
    }
}

__global__ void f32_to_bf16_kernel(const float* __restrict__ a, uint16_t* __restrict__ b, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        b[i] = f2bf(a[i]);
}

__global__ void bf16_to_f32_kernel(const uint16_t* __restrict__ a, float* __restrict__ b, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        b[i] = bf2f(a[i]);
}

// ------------------------------------------------------------ launchers

static unsigned grid_for(size_t n, unsigned block = 256, unsigned cap = 65536)
{
    size_t g = (n + block - 1) / block;
    if (g > cap) g = cap;
    if (g == 0) g = 1;
    return (unsigned)g;
}

struct FwdArgs {
    const uint16_t *in, *coarse;
    int Cc;
    const uint16_t* wt;
    const float* bias;
    uint16_t* out;
    int N, D, H, W, Cin, Cout, Kp, relu;
};

template <int NB, int QC, bool kPipe, int kMinWaves, int kAfter, bool kFlat = false>
static hipError_t launch_fwd(const FwdArgs& a, const FwdAfter& after, hipStream_t s)
{
    using T = FwdTile<NB, QC, kFlat>;
    const int cgroups = (a.Cout + 16 * NB - 1) / (16 * NB);
    dim3 grid((a.W + T::TX - 1) / T::TX, ((a.H + T::TY - 1) / T::TY) * cgroups, a.N * ((a.D + T::TZ - 1) / T::TZ));
    hipLaunchKernelGGL((conv3d_fwd_kernel<NB, QC, kPipe, kMinWaves, kAfter, kFlat>), grid, dim3(64 * T::WAVES), 0, s, a.in,
                       a.coarse, a.Cc, a.wt, a.bias, a.out, a.N, a.D, a.H, a.W, a.Cin, a.Cout, a.Kp, a.relu, after);
    return hipGetLastError();
}

template <int kAfter>
static hipError_t conv3d_fwd(const FwdArgs& a, const FwdAfter& after, hipStream_t s)
{
    const int N = a.N, D = a.D, H = a.H, W = a.W, Cin = a.Cin, Cout = a.Cout, Kp = a.Kp, Cc = a.Cc;
    if (Cin % 8 || Cin < 8 || Kp < 27 * Cin || Cc % 8 || Cc < 0 || Cc >= Cin || (Cc && !a.coarse) ||
        ((Cc || kAfter == kPool || kAfter == kSplit) && (D % 2 || H % 2 || W % 2)) || (kAfter == kHead && Cout != 16) ||
        (kAfter == kSplit && (after.Cc % 32 || after.Cc >= Cout)))
        return hipErrorInvalidValue;
    // the kernel keeps element offsets in 32 bits
    if ((size_t)N * D * H * W * (size_t)Cin >= (size_t)0x7FFFFFFF || (size_t)Cout * Kp >= (size_t)0x7FFFFFFF)
        return hipErrorInvalidValue;
    // Which tile, by what each was measured at (us; 160 x 128 x 128 voxels and
    // its halves; "1, 2" = the stage's chunks of 8 channels, "pipe" = two
    // buffers, one workgroup per CU):
    // - Up to 24 input channels there is little to gain from whole 32-byte
    //   pieces and the smaller buffers keep more workgroups resident:
    //   8 -> 16: 39 with 1, 59 with 2; 16 -> 48: 176 and 188.
    // - Grids of at most one workgroup per CU pipeline their stages:
    //   128 -> 64 at 20 x 16 x 16: 18.6 with pipe, 21.3 without; 64 -> 32 at
    //   40 x 32 x 32 (160 workgroups): 13.5 and 15.4; 32 -> 64 there (320
    //   workgroups): 15.4 and 11.3.
    // - Else two chunks and the resident workgroups overlap each other's
    //   copies: 48 -> 16: 153 with 2, 201 with 1 and pipe, 214 with 2 and pipe.
    //   32 output channels a workgroup where there are that many (32 -> 96:
    //   63 against 72 with 16; 48 -> 32 on 2 x 41 x 53 x 75: 45 and 53).
    const size_t tiles = (size_t)N * ((D + 3) / 4) * ((H + 7) / 8) * ((W + 15) / 16);
    const int n16 = (Cout + 15) / 16;
    // - One z plane wider than 16 voxels, more than one workgroup per CU: flat
    //   blocks, of which a quarter as many voxels lie outside: 48 -> 16 on 1024 x
    //   1024: 149 and 69; 32 -> 32 on 512 x 512: 53 and 23, on 2 x 100000: 123 and
    //   44; 64 -> 64 on 200 planes of 16 x 16: 44 and 52, so not there.  Two planes:
    //   48 -> 16 on 1024 x 1024: 170 and 346.
    if constexpr (kAfter == kPlain) {
        if (D == 1 && W > 16 && tiles * n16 > 256)
            return Cout <= 16 ? launch_fwd<1, 1, false, 8, kPlain, true>(a, after, s) : launch_fwd<2, 1, false, 6, kPlain, true>(a, after, s);
    }
    // (a stage of two chunks has one source and never runs past the last
    // channel; the network's head has 48 input channels, its other epilogues
    // 32 or more output channels where there are more than 24 input channels)
    if (Cin <= 24 || Cin % 16 || Cc % 16) {
        if constexpr (kAfter == kHead) return hipErrorInvalidValue;
        else return launch_fwd<1, 1, false, 8, kAfter>(a, after, s);
    }
    if (tiles * n16 <= 256) return launch_fwd<1, 2, true, 2, kAfter>(a, after, s);
    if constexpr (kAfter == kHead) {
        return launch_fwd<1, 2, false, 6, kAfter>(a, after, s);
    } else {
        if (kAfter == kPlain && Cout <= 16) return launch_fwd<1, 2, false, 6, kPlain>(a, after, s);
        return launch_fwd<2, 2, false, 4, kAfter>(a, after, s);
    }
}

hipError_t nn_conv3d_fwd(const uint16_t* in, const uint16_t* wt, const float* bias, uint16_t* out, int N,
                         int D, int H, int W, int Cin, int Cout, int Kp, int relu, hipStream_t s)
{
    return conv3d_fwd<kPlain>({in, nullptr, 0, wt, bias, out, N, D, H, W, Cin, Cout, Kp, relu}, {}, s);
}

hipError_t nn_conv3d_fwd_cat(const uint16_t* in, const uint16_t* coarse, int Cc, const uint16_t* wt,
                             const float* bias, uint16_t* out, int N, int D, int H, int W, int Cin, int Cout,
                             int Kp, int relu, hipStream_t s)
{
    return conv3d_fwd<kPlain>({in, coarse, Cc, wt, bias, out, N, D, H, W, Cin, Cout, Kp, relu}, {}, s);
}

hipError_t nn_conv3d_fwd_pool(const uint16_t* in, const uint16_t* wt, const float* bias, uint16_t* out,
                              uint16_t* pooled, int N, int D, int H, int W, int Cin, int Cout, int Kp, int relu,
                              hipStream_t s)
{
    FwdAfter after{};
    after.half = pooled;
    return conv3d_fwd<kPool>({in, nullptr, 0, wt, bias, out, N, D, H, W, Cin, Cout, Kp, relu}, after, s);
}

hipError_t nn_conv3d_fwd_split(const uint16_t* in, const uint16_t* wt, uint16_t* dcoarse, int Cc, uint16_t* dskip, int N,
                               int D, int H, int W, int Cin, int Cout, int Kp, hipStream_t s)
{
    FwdAfter after{};
    after.half = dcoarse;
    after.rest = dskip;
    after.Cc = Cc;
    return conv3d_fwd<kSplit>({in, nullptr, 0, wt, nullptr, nullptr, N, D, H, W, Cin, Cout, Kp, 0}, after, s);
}

// out (the rounded activations the head reads) may be NULL; d x h x wd: the
// caller's grid inside the network's
hipError_t nn_conv3d_fwd_cat_head(const uint16_t* in, const uint16_t* coarse, int Cc, const uint16_t* wt,
                                  const float* bias, uint16_t* out, const float* w, const float* b, const float* dose,
                                  const float* scale, float* res, int N, int D, int H, int W, int Cin, int Kp, int d,
                                  int h, int wd, hipStream_t s)
{
    FwdAfter after{};
    after.w = w;
    after.b = b;
    after.dose = dose;
    after.scale = scale;
    after.res = res;
    after.rg = Region{D, H, W, d, h, wd};
    return conv3d_fwd<kHead>({in, coarse, Cc, wt, bias, out, N, D, H, W, Cin, 16, Kp, 1}, after, s);
}

hipError_t nn_flip_weights(const FlipLayer* layers, int n, hipStream_t s)
{
    if (n < 1 || n > 7) return hipErrorInvalidValue;
    FlipLayers f{};
    int most = 0;
    for (int i = 0; i < n; ++i) {
        f.l[i] = layers[i];
        most = std::max(most, layers[i].Cin * layers[i].Kpf);
    }
    hipLaunchKernelGGL(flip_weights_kernel, dim3(grid_for(most), n), dim3(256), 0, s, f);
    return hipGetLastError();
}

template <int NCI, int NCO, bool kWide = false>
static hipError_t launch_wgrad(const uint16_t* in, const uint16_t* coarse, int Cc, const uint16_t* dout, float* dw, int N,
                               int D, int H, int W, int Cin, int Cout, int Kp, hipStream_t s)
{
    using T = WgTile<NCI, NCO>;
    const int n_xt = (W + 31) / 32, n_yt = (H + T::TY - 1) / T::TY;
    const int blocks = ((Cin + 16 * NCI - 1) / (16 * NCI)) * ((Cout + 16 * NCO - 1) / (16 * NCO));
    // one workgroup per CU (its waves fill it), the planes of a channel block
    // dealt to its workgroups in equal runs
    const unsigned long long n_planes = (unsigned long long)N * n_yt * n_xt * D;
    const int per_block = (int)std::min<unsigned long long>(n_planes, (unsigned long long)std::max(1, 256 / blocks));
    hipLaunchKernelGGL((conv3d_wgrad_kernel<NCI, NCO, kWide>), dim3((unsigned)(blocks * per_block)), dim3(64 * kWgWaves), 0, s, in,
                       coarse, Cc, dout, dw, D, H, W, Cin, Cout, Kp, n_xt, n_yt, n_planes, per_block);
    return hipGetLastError();
}

hipError_t nn_conv3d_wgrad_cat(const uint16_t* in, const uint16_t* coarse, int Cc, const uint16_t* dout, float* dw, int N,
                               int D, int H, int W, int Cin, int Cout, int Kp, hipStream_t s)
{
    if (Cc < 0 || Cc % 16 || Cc >= Cin || (Cc && !coarse) || (Cc && (D % 2 || H % 2 || W % 2))) return hipErrorInvalidValue;
#define PMC_WG(NCI, ...) launch_wgrad<NCI, __VA_ARGS__>(in, coarse, Cc, dout, dw, N, D, H, W, Cin, Cout, Kp, s)
    // z planes of 4 GiB and more (2^28 voxels of 8 channels): past the 32-bit
    // byte offsets; one tiling serves them, bound by the planes' bytes
    if ((size_t)H * W * (size_t)std::max(Cin, Cout) >= (size_t)0x7FFFFFFF) return PMC_WG(2, 2, true);
    // input tiles: three of 16 channels where they divide the channels, else two, or one
    const int ti = (Cin + 15) / 16, to = (Cout + 15) / 16;
    const int nci = ti % 3 == 0 ? 3 : (ti == 1 ? 1 : 2);
    if (to == 1) return nci == 3 ? PMC_WG(3, 1) : (nci == 2 ? PMC_WG(2, 1) : PMC_WG(1, 1));
    return nci == 3 ? PMC_WG(3, 2) : (nci == 2 ? PMC_WG(2, 2) : PMC_WG(1, 2));
#undef PMC_WG
}

hipError_t nn_conv3d_wgrad(const uint16_t* in, const uint16_t* dout, float* dw, int N, int D, int H, int W,
                           int Cin, int Cout, int Kp, hipStream_t s)
{
    return nn_conv3d_wgrad_cat(in, nullptr, 0, dout, dw, N, D, H, W, Cin, Cout, Kp, s);
}

// dpool NULL: no pooled output's gradient to add
hipError_t nn_grad_relu(const uint16_t* src, const uint16_t* dpool, const uint16_t* y, uint16_t* dy, float* db, int N,
                        int D, int H, int W, int C, hipStream_t s)
{
    if (C < 8 || C > 256 || C % 8 || 256 % (C / 8) || (dpool && (D % 2 || H % 2 || W % 2))) return hipErrorInvalidValue;
    const unsigned rows = (unsigned)N * D * H;
    const unsigned blocks = std::min(512u, std::max(1u, rows / 4));
    if (dpool)
        hipLaunchKernelGGL(grad_relu_kernel<true>, dim3(blocks), dim3(256), 0, s, src, dpool, y, dy, db, rows, D, H, W, C);
    else
        hipLaunchKernelGGL(grad_relu_kernel<false>, dim3(blocks), dim3(256), 0, s, src, dpool, y, dy, db, rows, D, H, W, C);
    return hipGetLastError();
}

// scale: 1 + kParts floats, the first the maximum dose; nvox: voxels of the
// network grid; the region gives the caller's (compact)
// grid inside it, whose ncomp = n d h w voxels hold dose and density
hipError_t nn_make_input(const float* dose, const float* rho, float* scale, uint16_t* x, size_t nvox, int N, int D,
                         int H, int W, int d, int h, int w, hipStream_t s)
{
    const Region rg{D, H, W, d, h, w};
    const size_t ncomp = (size_t)N * d * h * w;
    const unsigned parts = grid_for(ncomp, 256, kParts);
    hipLaunchKernelGGL(max_kernel, dim3(parts), dim3(256), 0, s, dose, ncomp, scale + 1);
    hipLaunchKernelGGL(make_input_kernel, dim3(grid_for(nvox, 256, 2048)), dim3(256), 0, s, dose, rho, scale, (int)parts,
                       reinterpret_cast<uint4*>(x), nvox, rg);
    return hipGetLastError();
}

// region_part: kParts counts (device); loss_part: the shares of the loss
// (pinned host memory, up to 2 kParts), of which *n_loss are written
hipError_t nn_loss_head_bwd(const float* out, const float* target, const float* dose, const float* scale,
                            unsigned int* region_part, const uint16_t* d1, const float* w, uint16_t* dd1, float* dw,
                            float* db, float* dbias, double* loss_part, int* n_loss, size_t nvox, hipStream_t s)
{
    const unsigned blocks = grid_for(nvox, 256, kParts);
    hipLaunchKernelGGL(region_count_kernel, dim3(blocks), dim3(256), 0, s, dose, nvox, scale, 0.01f, region_part);
    *n_loss = (int)grid_for(nvox, 256, 2 * kParts);
    hipLaunchKernelGGL(loss_head_bwd_kernel, dim3(*n_loss), dim3(256), 0, s, out, target, scale, d1, w, dd1, dw, db, dbias,
                       loss_part, nvox, (const unsigned int*)region_part, (int)blocks);
    return hipGetLastError();
}

hipError_t nn_adam(float* p, float* g, float* m1, float* m2, uint16_t* p_bf, size_t n, float lr, float b1, float b2,
                   float eps, float c1, float c2, float gs, hipStream_t s)
{
    hipLaunchKernelGGL(adam_kernel, dim3(grid_for(n)), dim3(256), 0, s, p, g, m1, m2, p_bf, n, lr, b1, b2, eps, c1, c2,
                       gs);
    return hipGetLastError();
}

// parts: kParts shares (pinned host memory), of which *n_parts are written
hipError_t nn_sqnorm(const float* g, size_t n, double* parts, int* n_parts, hipStream_t s)
{
    *n_parts = (int)grid_for(n, 256, kParts);
    hipLaunchKernelGGL(sqnorm_kernel, dim3(*n_parts), dim3(256), 0, s, g, n, parts);
    return hipGetLastError();
}

hipError_t nn_f32_to_bf16(const float* a, uint16_t* b, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(f32_to_bf16_kernel, dim3(grid_for(n)), dim3(256), 0, s, a, b, n);
    return hipGetLastError();
}

// Matrix-core throughput probe: every wave issues `iters` rounds of eight
// independent v_mfma_f32_16x16x32_bf16 on register operands (no memory
// traffic in the loop); the accumulators are written out once so that the
// work stays live.  16,384 FLOP per instruction.  The instructions are
// written out so that each accumulates in place: from the builtin the
// register allocator rotated the eight accumulators through other registers
// every iteration (about 18 register moves per 8 MFMAs), which measured the
// moves, not the matrix cores.
__global__ void __launch_bounds__(256) mfma_probe_kernel(int iters, float* __restrict__ sink)
{
    const int lane = threadIdx.x & 63;
    bf16x8 a, b;
    for (int i = 0; i < 8; ++i) {
        a[i] = (__bf16)(0.001f * (float)(lane + i));
        b[i] = (__bf16)(0.002f * (float)(lane - i));
    }
    f32x4 acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int k = 0; k < 8; ++k)
            asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[k]) : "v"(a), "v"(b));
    }
    // the compiler does not track these instructions' results: wait out the
    // last MFMA's passes before the accumulators are read (the accumulators
    // pass through the wait, so no read is scheduled ahead of it)
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7"
                 : "+a"(acc[0]), "+a"(acc[1]), "+a"(acc[2]), "+a"(acc[3]), "+a"(acc[4]), "+a"(acc[5]),
                   "+a"(acc[6]), "+a"(acc[7]));
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) t += acc[k][0] + acc[k][1] + acc[k][2] + acc[k][3];
    sink[blockIdx.x * blockDim.x + threadIdx.x] = t;
}

hipError_t nn_mfma_probe(int grid, int iters, float* sink, hipStream_t s)
{
    hipLaunchKernelGGL(mfma_probe_kernel, dim3(grid), dim3(256), 0, s, iters, sink);
    return hipGetLastError();
}

hipError_t nn_bf16_to_f32(const uint16_t* a, float* b, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(bf16_to_f32_kernel, dim3(grid_for(n)), dim3(256), 0, s, a, b, n);
    return hipGetLastError();
}

}  // namespace pmc
