// BF16-MFMA / FP32-accumulate kernels of the grid U-Net surrogate (gfx950).
//
// Activations are BF16, channels-last [N][D][H][W][C]; a kernel reads or
// writes a channel slice [off, off + cnt) of a tensor with channel stride C,
// so skip concatenation costs nothing.  Channel counts used by the MFMA
// paths are multiples of 16.
//
// Convolution = implicit GEMM on the BF16 MFMAs:
//   forward  D[voxel][co] = sum_{tap, ci} X[p(voxel, tap)][ci] W[tap][ci][co]
//   dgrad    the same kernel on dY with flipped, transposed weights
//   wgrad    D[ci][co] += sum_voxel X[p(voxel, tap)][ci] dY[voxel][co]
// with tap geometries: 3^3 zero-padded ("c3"), 3^3 over a nearest x2
// upsampled input ("up"), 2^3 stride 2 ("down") and 1^3 ("c1").  The 3^3
// kinds with a multiple of 32 input channels, the 3^3 first layer over 8
// channels and every weight gradient run on v_mfma_f32_16x16x32_bf16
// (gfx950, twice the rate of the 16x16x16 form); the rest on
// v_mfma_f32_16x16x16bf16_1k.
// Operand lane layout (wave64, 16x16x16): A[i][k] sits in lane i + 16 (k/4),
// element k % 4; B[k][j] in lane j + 16 (k/4), element k % 4; D[i][j] in lane
// j + 16 (i/4), element i % 4.  16x16x32: A[i][k] in lane i + 16 (k/8),
// element k % 8; B[k][j] in lane j + 16 (k/8), element k % 8; D as above.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nn_kernels.hpp"
#include "nn_plan.hpp"

namespace nn {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffff) ? 0x40 : 0));   // inf / nan
    u += 0x7fffu + ((u >> 16) & 1u);                                                                 // nearest even
    return (uint16_t)(u >> 16);
}

// Two of them packed (v_cvt_pk_bf16_f32 rounds to nearest even and keeps infinities and NaN).
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi)
{
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, b2{(__bf16)lo, (__bf16)hi});
}

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ int ksize(int kind) { return kind == KIND_C3 || kind == KIND_UP ? 3 : (kind == KIND_DOWN ? 2 : 1); }

// Input voxel read by output voxel (z, y, x) through tap (a, b, c); false if
// it lies in the zero padding.  (D, H, W) are the input's spatial sizes.
__device__ __forceinline__ bool tap_source(int kind, int z, int y, int x, int a, int b, int c, int D, int H, int W,
                                           int &sz, int &sy, int &sx)
{
    if (kind == KIND_C3) {
        sz = z + a - 1; sy = y + b - 1; sx = x + c - 1;
        return sz >= 0 && sy >= 0 && sx >= 0 && sz < D && sy < H && sx < W;
    }
    if (kind == KIND_UP) {
        int uz = z + a - 1, uy = y + b - 1, ux = x + c - 1;
        if (uz < 0 || uy < 0 || ux < 0 || uz >= 2 * D || uy >= 2 * H || ux >= 2 * W) return false;
        sz = uz >> 1; sy = uy >> 1; sx = ux >> 1;
        return true;
    }
    if (kind == KIND_DOWN) {
        sz = 2 * z + a; sy = 2 * y + b; sx = 2 * x + c;
        return true;
    }
    sz = z; sy = y; sx = x;
    return true;
}

// Four consecutive channels co .. co + 3 of output voxel v (bias and ReLU applied here).
__device__ __forceinline__ void store4(const ConvArgs &a, long long v, int co, const f4 acc, const float bias[4], bool y8)
{
    float val[4];
#pragma unroll
    for (int r = 0; r < 4; r++) {
        val[r] = acc[r] + bias[r];
        if (a.relu) val[r] = fmaxf(val[r], 0.0f);
    }
    if (a.y) {
        uint16_t *yp = a.y + v * a.cy + a.y_off + co;
        if (y8 && co + 4 <= a.cout) {
            *(uint2 *)yp = make_uint2(f2bf2(val[0], val[1]), f2bf2(val[2], val[3]));
        } else {
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (co + r < a.cout) yp[r] = f2bf(val[r]);
        }
    }
    if (a.y32) {
        float *yp = a.y32 + v * a.cy32 + co;
        if (co + 4 <= a.cout && a.cy32 % 4 == 0 && ((uintptr_t)a.y32 & 15) == 0) {
            *(float4 *)yp = make_float4(val[0], val[1], val[2], val[3]);
        } else {
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (co + r < a.cout) yp[r] = val[r];
        }
    }
}

// Whether a BF16 output slice takes 8-byte stores of four channels.
__device__ __forceinline__ bool stores8(const ConvArgs &a)
{
    return a.cy % 4 == 0 && a.y_off % 4 == 0 && ((uintptr_t)a.y & 7) == 0;
}

__device__ __forceinline__ void load_bias4(const ConvArgs &a, int co, float bias[4])
{
#pragma unroll
    for (int r = 0; r < 4; r++) bias[r] = a.bias && co + r < a.cout ? a.bias[co + r] : 0.0f;
}

// ---------------------------------------------------------------- convolution without halo reuse (2^3 stride 2, 1^3)
// One wave computes 16 MF consecutive output voxels x 16 NF output channels
// (block cg of ncg; the waves of a workgroup share the voxels' lines).  Each
// input voxel meets one tap, so the fragments come straight from memory, and
// what bounds the kernel is fetching their lines: a load takes 32 of a voxel's
// bytes (the order of the sum is that of 16-channel chunks), so a wave covers
// up to 64 output channels before another reads them again, and small grids
// take fewer voxels per wave.  The weights are the MFMA's row operand (8-byte
// stores).  Measured on 64 boxes of 40 x 24 x 40 (us, one wave per 64 voxels
// and 2-byte stores before): stride 2 32 -> 64 104 (126), 64 -> 128 46 (86),
// 1^3 head 52 (67).
template <int MF, int NF, int KC>
__global__ __launch_bounds__(256) void k_conv(ConvArgs a, int ncg)
{
    const int lane = threadIdx.x & 63;
    const long long wave = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const long long nvox = (long long)a.n * a.od * a.oh * a.ow;
    const int cg = (int)(wave % ncg);
    const long long v0 = wave / ncg * (16 * MF);
    if (v0 >= nvox) return;
    const int ks = ksize(a.kind);
    const int ntap = ks * ks * ks;
    const int kc = KC ? KC : a.cin / 16, nft = (a.cout + 15) / 16, cn = cg * NF;
    f4 acc[MF][NF];
#pragma unroll
    for (int f = 0; f < MF; f++)
#pragma unroll
        for (int n = 0; n < NF; n++) acc[f][n] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    // first input voxel of this lane's output voxels (one per fragment); past the end: the last voxel again
    const int g = lane >> 4, i = lane & 15;
    const uint16_t *src[MF];
#pragma unroll
    for (int f = 0; f < MF; f++) {
        const long long v = min(v0 + 16 * f + i, nvox - 1);
        const int x = (int)(v % a.ow);
        long long r = v / a.ow;
        const int y = (int)(r % a.oh);
        r /= a.oh;
        const int z = (int)(r % a.od), nn = (int)(r / a.od);
        src[f] = a.x + (((((long long)nn * a.id + ks * z) * a.ih + ks * y) * a.iw + ks * x) * a.cx + a.x_off + 4 * g);
    }
    const uint16_t *w = a.w + (size_t)cn * 256 + 4 * lane;
    for (int t = 0; t < ntap; t++) {
        const long long off = (((long long)(t / (ks * ks)) * a.ih + (t / ks) % ks) * a.iw + t % ks) * a.cx;
#pragma unroll KC ? KC : 1
        for (int c = 0; c < kc; c++) {
            s4 A[MF];
#pragma unroll
            for (int f = 0; f < MF; f++) A[f] = __builtin_bit_cast(s4, *(const uint2 *)(src[f] + off + 16 * c));
#pragma unroll
            for (int n = 0; n < NF; n++) {
                const s4 Bv = __builtin_bit_cast(s4, *(const uint2 *)(w + ((size_t)(t * kc + c) * nft + n) * 256));
#pragma unroll
                for (int f = 0; f < MF; f++) acc[f][n] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(Bv, A[f], acc[f][n], 0, 0, 0);
            }
        }
    }
    // D[row][col]: channel 16 (cn + n) + 4 g + r of voxel v0 + 16 f + i
    const bool y8 = stores8(a);
#pragma unroll
    for (int n = 0; n < NF; n++) {
        const int co = 16 * (cn + n) + 4 * g;
        float bias[4];
        load_bias4(a, co, bias);
#pragma unroll
        for (int f = 0; f < MF; f++)
            if (v0 + 16 * f + i < nvox) store4(a, v0 + 16 * f + i, co, acc[f][n], bias, y8);
    }
}

// ---------------------------------------------------------------- LDS-tiled convolution (3^3 and up)
// A workgroup computes a 4 x 4 x 16 (z, y, x) tile of output voxels for all
// output channels; wave w owns the z-slice w (4 row fragments of 16 x).  For
// every 16-channel chunk of the input, the tile's input halo is staged once
// in LDS (zero where the padding or the tensor edge is) and all 27 taps read
// their A fragments from it; weights come from the packed B fragments.
constexpr int TLZ = 4, TLY = 4, TLX = 16;
constexpr int HLZ = TLZ + 2, HLY = TLY + 2, HLX = TLX + 2;   // 3^3 halo (the up halo is smaller)

template <int NF, int KIND>
__global__ __launch_bounds__(256) void k_conv_lds(ConvArgs a)
{
    __shared__ uint2 halo[HLZ * HLY * HLX * 4];              // [voxel][4 x (4 bf16)]
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int tiles_x = (a.ow + TLX - 1) / TLX, tiles_y = (a.oh + TLY - 1) / TLY, tiles_z = (a.od + TLZ - 1) / TLZ;
    int b = blockIdx.x;
    const int bx = b % tiles_x;
    b /= tiles_x;
    const int by = b % tiles_y;
    b /= tiles_y;
    const int bz = b % tiles_z;
    const int bn = b / tiles_z;
    const int z0 = bz * TLZ, y0 = by * TLY, x0 = bx * TLX;
    // input-space origin and extent of the halo
    int hz0, hy0, hx0, hz, hy, hx;
    if (KIND == KIND_C3) {
        hz0 = z0 - 1; hy0 = y0 - 1; hx0 = x0 - 1;
        hz = HLZ; hy = HLY; hx = HLX;
    } else {   // nearest x2 upsampled input: fine u = o + t - 1 reads coarse u >> 1
        hz0 = (z0 >> 1) - 1; hy0 = (y0 >> 1) - 1; hx0 = (x0 >> 1) - 1;
        hz = TLZ / 2 + 2; hy = TLY / 2 + 2; hx = TLX / 2 + 2;
    }
    const int nh = hz * hy * hx;
    f4 acc[4][NF];
#pragma unroll
    for (int f = 0; f < 4; f++)
#pragma unroll
        for (int n = 0; n < NF; n++) acc[f][n] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    const int kc = a.cin / 16;
    const int q = lane >> 4, i = lane & 15;
    for (int c = 0; c < kc; c++) {
        // stage the halo of input channels [16 c, 16 c + 16)
        for (int e = threadIdx.x; e < nh * 4; e += 256) {
            const int v = e >> 2, qq = e & 3;
            const int lx = v % hx, ly = (v / hx) % hy, lz = v / (hx * hy);
            const int gz = hz0 + lz, gy = hy0 + ly, gx = hx0 + lx;
            uint2 val = make_uint2(0u, 0u);
            if (gz >= 0 && gy >= 0 && gx >= 0 && gz < a.id && gy < a.ih && gx < a.iw)
                val = *(const uint2 *)(a.x + ((((long long)bn * a.id + gz) * a.ih + gy) * a.iw + gx) * a.cx + a.x_off +
                                       16 * c + 4 * qq);
            halo[e] = val;
        }
        __syncthreads();
        const uint16_t *wc = a.w + (size_t)c * NF * 256 + 4 * lane;
        for (int t = 0; t < 27; t++) {
            const int ta = t / 9, tb = (t / 3) % 3, tc = t % 3;
            s4 Af[4];
#pragma unroll
            for (int f = 0; f < 4; f++) {
                int lz, ly, lx;
                if (KIND == KIND_C3) {
                    lz = wv + ta; ly = f + tb; lx = i + tc;
                } else {
                    lz = ((z0 + wv + ta - 1) >> 1) - hz0;
                    ly = ((y0 + f + tb - 1) >> 1) - hy0;
                    lx = ((x0 + i + tc - 1) >> 1) - hx0;
                }
                const uint2 raw = halo[((lz * hy + ly) * hx + lx) * 4 + q];
                Af[f] = s4{(short)(raw.x & 0xffff), (short)(raw.x >> 16), (short)(raw.y & 0xffff), (short)(raw.y >> 16)};
            }
            const uint16_t *wt = wc + (size_t)t * kc * NF * 256;
#pragma unroll
            for (int n = 0; n < NF; n++) {
                const uint2 raw = *(const uint2 *)(wt + (size_t)n * 256);
                const s4 Bv = s4{(short)(raw.x & 0xffff), (short)(raw.x >> 16), (short)(raw.y & 0xffff), (short)(raw.y >> 16)};
#pragma unroll
                for (int f = 0; f < 4; f++) acc[f][n] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(Af[f], Bv, acc[f][n], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    // epilogue: fragment f = output row y0 + f, D[i][j] -> x = x0 + 4 (lane/16) + r, channel 16 n + lane % 16
    const int oz = z0 + wv;
#pragma unroll
    for (int f = 0; f < 4; f++) {
        const int oy = y0 + f;
        if (oz >= a.od || oy >= a.oh) continue;
#pragma unroll
        for (int n = 0; n < NF; n++) {
            const int co = 16 * n + (lane & 15);
            if (co >= a.cout) continue;
            const float bias = a.bias ? a.bias[co] : 0.0f;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int ox = x0 + 4 * (lane >> 4) + r;
                if (ox >= a.ow) continue;
                const long long v = (((long long)bn * a.od + oz) * a.oh + oy) * a.ow + ox;
                float val = acc[f][n][r] + bias;
                if (a.relu) val = fmaxf(val, 0.0f);
                if (a.y) a.y[v * a.cy + a.y_off + co] = f2bf(val);
                if (a.y32) a.y32[v * a.cy32 + co] = val;
            }
        }
    }
}

typedef __bf16 b8 __attribute__((ext_vector_type(8)));

__device__ __align__(16) uint16_t g_zero_piece[8];   // 16 zero bytes: the source of padding voxels

// floor(v / d) by the reciprocal ceil(2^32 / d), v < 2^16.
__device__ __forceinline__ int div_by(unsigned v, unsigned magic, int d) { return d == 1 ? (int)v : (int)__umulhi(v, magic); }

// 8 channels of a tensor row that cannot be copied as 16 aligned bytes; channels past n are zero.
__device__ __forceinline__ uint4 load_piece(const uint16_t *p, int n)
{
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < 8; k++)
        if (k < n) w[k >> 1] |= (uint32_t)p[k] << (16 * (k & 1));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// 3^3 and upsampling convolution on v_mfma_f32_16x16x32_bf16 for a multiple of
// 32 input channels.  K slot e of lane group g (= lane / 16) carries channel
// 8 g + e of the 32-channel chunk, for A (halo) and B (packed weights) alike.
//
// A workgroup computes a tile of TZ x FR x TX (z, y, x) output voxels.  The 16
// rows of an A fragment are any 16 positions of the tile's (z, x) plane at one
// y (each lane keeps the halo offsets of its position), so a tile can be cut
// to the grid instead of to 4 x 16: on the 40 x 24 x 40, 20 x 12 x 20 and
// 10 x 6 x 10 levels of a 40 x 24 x 40 box 4 x 4 x 16 tiles spend 17, 37 and
// 61 % of the MFMAs on padding.  Wave (pw, cw) owns positions 16 pw .. + 15,
// all FR rows and output channels 16 NF (cw + ...) .. + 16 NF - 1.  For each
// (z tap, x tap) it reads the FR + 2 halo rows its FR output rows see through
// the three y taps once; every B fragment (weights, through the vector cache)
// feeds FR MFMAs, so that at FR = 8 and NF = 2 neither the LDS (53 of 128
// bytes per clock at the MFMA rate) nor the vector cache (31 of 64) bounds it.
// The halo holds, per voxel, the chunk's four 16-byte pieces (channels
// 8 p .. 8 p + 7), piece p at slot p ^ ((x >> 2) & 3) so that the reads of 8
// neighbouring voxels hit distinct banks.  It is staged by 16-byte
// global-to-LDS copies, every load of a chunk in flight at once; voxels in the
// padding copy from a zero block.  The weights are the MFMA's row operand, so
// that a lane ends with four consecutive channels of one voxel and stores
// them as 8 bytes (through LDS, as 16-byte rows, the epilogue took a third of
// a 32 -> 32 layer).  The order of the sum (channel chunk, z tap, x tap,
// y tap) does not depend on the tile.  Measured on 64 boxes of 40 x 24 x 40
// (us, 4 x 4 or 4 x 8 x 16 tiles before): 32 -> 32 141 (235), 64 -> 32 262 (430),
// 64 -> 64 at half size 61 (147), 128 -> 128 at quarter size 37 (190),
// upsampling 64 -> 32 167 (314) and 128 -> 64 98 (231).
template <int NF, int KIND, int FR>
__global__ __launch_bounds__((NF == 2 && FR == 8 ? 8 : 16) * 64) void k_conv_pos(ConvArgs a, ConvPlan p)
{
    typedef __attribute__((address_space(3))) void lds_void;
    typedef const __attribute__((address_space(1))) void glob_void;
    extern __shared__ uint4 halo[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nt = 64 * p.PW * p.CW;
    // every XCD takes a run of neighbouring tiles (their halos overlap in its L2), and the
    // output-channel blocks of one tile run on one XCD at about the same time
    const int q8 = blockIdx.x >> 3;
    const int per = (p.ntiles + 7) >> 3;
    const int tile = (blockIdx.x & 7) * per + q8 / p.nco;
    if (q8 / p.nco >= per || tile >= p.ntiles) return;
    const int pw = wv % p.PW, cn = (q8 % p.nco * p.CW + wv / p.PW) * NF;   // first output fragment
    int b = tile;
    const int x0 = (b % p.tiles_x) * p.TX;
    b /= p.tiles_x;
    const int y0 = (b % p.tiles_y) * FR;
    b /= p.tiles_y;
    const int z0 = (b % p.tiles_z) * p.TZ, bn = b / p.tiles_z;
    int hz0, hy0, hx0;
    if (KIND == KIND_C3) {
        hz0 = z0 - 1; hy0 = y0 - 1; hx0 = x0 - 1;
    } else {   // nearest x2 upsampled input: fine u = o + t - 1 reads coarse u >> 1
        hz0 = (z0 - 1) >> 1; hy0 = (y0 - 1) >> 1; hx0 = (x0 - 1) >> 1;
    }
    const int g = lane >> 4, i = lane & 15;
    const int pos = 16 * pw + i, nreal = p.TZ * p.TX;
    const int pz = pos < nreal ? div_by(pos, p.mTX, p.TX) : 0, px = pos < nreal ? pos - pz * p.TX : 0;
    const int hrow = 64 * p.HX;                           // bytes of a halo row
    int zo[3], xo[3];                                     // halo byte offsets of this lane per z and x tap
#pragma unroll
    for (int t = 0; t < 3; t++) {
        zo[t] = (KIND == KIND_C3 ? pz + t : ((z0 + pz + t - 1) >> 1) - hz0) * p.HY * hrow;
        const int lx = KIND == KIND_C3 ? px + t : ((x0 + px + t - 1) >> 1) - hx0;
        xo[t] = 64 * lx + 16 * (g ^ ((lx >> 2) & 3));
    }
    f4 acc[FR][NF];
#pragma unroll
    for (int f = 0; f < FR; f++)
#pragma unroll
        for (int n = 0; n < NF; n++) acc[f][n] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    const int kc = a.cin / 32, nft = (a.cout + 15) / 16, ns = 4 * p.HZ * p.HY * p.HX;
    const VoxelIndex xi(a.ih, a.iw, a.cx, p.wide);
    const uint16_t *xb = a.x + (size_t)bn * a.id * a.ih * a.iw * a.cx + a.x_off;
    for (int c = 0; c < kc; c++) {
        for (int s0 = 64 * wv; s0 < ns; s0 += nt) {
            const int s = s0 + lane;
            if (s >= ns) break;
            const int v = s >> 2;
            const int q = div_by(v, p.mHX, p.HX), lx = v - q * p.HX, lz = div_by(q, p.mHY, p.HY), ly = q - lz * p.HY;
            const int c8 = 8 * ((s & 3) ^ ((lx >> 2) & 3));
            const int gz = hz0 + lz, gy = hy0 + ly, gx = hx0 + lx;
            const bool in = gz >= 0 && gy >= 0 && gx >= 0 && gz < a.id && gy < a.ih && gx < a.iw;
            const uint16_t *src =
                in ? xb + xi(gz, gy, gx) + 32 * c + c8 : g_zero_piece;
            if (p.x16) __builtin_amdgcn_global_load_lds((glob_void *)src, (lds_void *)(halo + s0), 16, 0, 0);
            else halo[s] = load_piece(src, 8);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the copies are not tracked by the compiler
        __syncthreads();
        const uint16_t *wc = a.w + ((size_t)c * nft + cn) * 512 + 8 * lane;
        const size_t wt = (size_t)kc * nft * 512;          // from one tap to the next
#pragma unroll 1
        for (int ta = 0; ta < 3; ta++) {
#pragma unroll 1
            for (int tc = 0; tc < 3; tc++) {
                const int v0 = (ta == 0 ? zo[0] : (ta == 1 ? zo[1] : zo[2])) + (tc == 0 ? xo[0] : (tc == 1 ? xo[1] : xo[2]));
                const uint16_t *w = wc + (ta * 9 + tc) * wt;
                b8 Bv[3][NF];
#pragma unroll
                for (int tb = 0; tb < 3; tb++)
#pragma unroll
                    for (int n = 0; n < NF; n++) Bv[tb][n] = __builtin_bit_cast(b8, *(const uint4 *)(w + 3 * tb * wt + n * 512));
                b8 Ar[FR + 2];
#pragma unroll
                for (int r = 0; r < FR + 2; r++) {
                    const int ly = KIND == KIND_C3 ? r : (r + 1) >> 1;   // y0 is even
                    Ar[r] = __builtin_bit_cast(b8, *(const uint4 *)((const char *)halo + (v0 + ly * hrow)));
                }
#pragma unroll
                for (int tb = 0; tb < 3; tb++)
#pragma unroll
                    for (int n = 0; n < NF; n++)
#pragma unroll
                        for (int f = 0; f < FR; f++)
                            acc[f][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Bv[tb][n], Ar[f + tb], acc[f][n], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    // D[row][col]: channel 16 (cn + n) + 4 g + r of position i
    const int gz = z0 + pz, gx = x0 + px;
    if (pos >= nreal || gz >= a.od || gx >= a.ow) return;
    float bias[NF][4];
#pragma unroll
    for (int n = 0; n < NF; n++) load_bias4(a, 16 * (cn + n) + 4 * g, bias[n]);
    const bool y8 = stores8(a);
#pragma unroll
    for (int f = 0; f < FR; f++) {
        if (y0 + f >= a.oh) break;
        const long long v = (((long long)bn * a.od + gz) * a.oh + y0 + f) * a.ow + gx;
#pragma unroll
        for (int n = 0; n < NF; n++) store4(a, v, 16 * (cn + n) + 4 * g, acc[f][n], bias[n], y8);
    }
}

// First layer: 3^3 convolution over 8 input channels with the taps folded
// into K.  K step c (32 wide) covers taps 4 c .. 4 c + 3: lane group g takes
// tap 4 c + g and its 8 elements are the 8 channels of that tap's input voxel
// (one 16-byte LDS read); 7 steps cover the 27 taps (the 28th has zero
// weights and reads tap 26's voxel).  The halo holds 8 channels per voxel.
// Tiles as k_conv_pos (four waves of 16 positions, 4 rows, all channels); memory
// bounds it (235 MB on 64 boxes of 40 x 24 x 40 in 88 us).
constexpr int FIRST_STEPS = 7;

template <int NF>
__global__ __launch_bounds__(256) void k_conv_first(ConvArgs a, ConvPlan p)
{
    typedef __attribute__((address_space(3))) void lds_void;
    typedef const __attribute__((address_space(1))) void glob_void;
    constexpr int FR = FIRST_ROWS, HY = FR + 2;
    extern __shared__ uint4 halo[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int per = (p.ntiles + 7) >> 3, tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || tile >= p.ntiles) return;
    int b = tile;
    const int x0 = (b % p.tiles_x) * p.TX;
    b /= p.tiles_x;
    const int y0 = (b % p.tiles_y) * FR;
    b /= p.tiles_y;
    const int z0 = (b % p.tiles_z) * p.TZ, bn = b / p.tiles_z;
    const VoxelIndex xi(a.ih, a.iw, a.cx, p.wide);
    const uint16_t *xb = a.x + (size_t)bn * a.id * a.ih * a.iw * a.cx + a.x_off;
    const int nh = p.HZ * HY * p.HX;
    for (int s0 = 64 * wv; s0 < nh; s0 += 256) {
        const int v = s0 + lane;
        if (v >= nh) break;
        const int q = div_by(v, p.mHX, p.HX), lx = v - q * p.HX, lz = q / HY, ly = q - lz * HY;
        const int gz = z0 - 1 + lz, gy = y0 - 1 + ly, gx = x0 - 1 + lx;
        const bool in = gz >= 0 && gy >= 0 && gx >= 0 && gz < a.id && gy < a.ih && gx < a.iw;
        const uint16_t *src = in ? xb + xi(gz, gy, gx) : g_zero_piece;
        __builtin_amdgcn_global_load_lds((glob_void *)src, (lds_void *)(halo + s0), 16, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the copies are not tracked by the compiler
    __syncthreads();
    f4 acc[FR][NF];
#pragma unroll
    for (int f = 0; f < FR; f++)
#pragma unroll
        for (int n = 0; n < NF; n++) acc[f][n] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    const int g = lane >> 4, i = lane & 15;
    const int pos = 16 * wv + i, nreal = p.TZ * p.TX;
    const int pz = pos < nreal ? div_by(pos, p.mTX, p.TX) : 0, px = pos < nreal ? pos - pz * p.TX : 0;
    const int base = pz * HY * p.HX + px;
#pragma unroll
    for (int c = 0; c < FIRST_STEPS; c++) {
        const int t = min(4 * c + g, 26);
        const int ta = t / 9, tb = (t / 3) % 3, tc = t % 3;
        b8 A[FR];
#pragma unroll
        for (int f = 0; f < FR; f++) A[f] = __builtin_bit_cast(b8, halo[base + (ta * HY + f + tb) * p.HX + tc]);
#pragma unroll
        for (int n = 0; n < NF; n++) {
            const b8 Bv = __builtin_bit_cast(b8, *(const uint4 *)(a.w + ((size_t)(c * NF + n) * 64 + lane) * 8));
#pragma unroll
            for (int f = 0; f < FR; f++) acc[f][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Bv, A[f], acc[f][n], 0, 0, 0);
        }
    }
    const int gz = z0 + pz, gx = x0 + px;
    if (pos >= nreal || gz >= a.od || gx >= a.ow) return;
    const bool y8 = stores8(a);
#pragma unroll
    for (int n = 0; n < NF; n++) {
        float bias[4];
        load_bias4(a, 16 * n + 4 * g, bias);
#pragma unroll
        for (int f = 0; f < FR; f++)
            if (y0 + f < a.oh)
                store4(a, (((long long)bn * a.od + gz) * a.oh + y0 + f) * a.ow + gx, 16 * n + 4 * g, acc[f][n], bias, y8);
    }
}

// Pack FP32 master weights W[tap][ci][co] (ci < cin, co < cout) into the
// B-fragment order the conv kernel reads, as BF16; `transpose` packs the
// weights of the adjoint (dgrad) convolution: taps mirrored, ci <-> co.
//   k32 = 0: element (((t * KC + c) * NF + n) * 64 + lane) * 4 + r holds
//            B[k][j], k = 16 c + 4 (lane / 16) + r (16x16x16 fragments);
//   k32 = 1: element (((t * KC2 + c) * NF + n) * 64 + lane) * 8 + e holds
//            k = 32 c + 8 (lane / 16) + e (16x16x32 fragments).
//   k32 = 2: the first-layer order (8 input channels, taps folded into K):
//            element ((c * NF + n) * 64 + lane) * 8 + j holds tap 4 c + lane / 16
//            (zero for tap 27), channel j.
// The job of this workgroup: one comparison per lane.
template <class Job>
__device__ __forceinline__ int job_of(const Jobs<Job> &q)
{
    const int l = threadIdx.x & 63;
    return __popcll(__ballot(l < q.count && (int)blockIdx.x >= q.first[l])) - 1;
}

// Threads take four elements in a row (one lane's fragment, or half of it) of
// 1,024 per workgroup.  All the tensors of a network go into one launch: a
// parameter update is bound by its launches, not by its 60 MB (see k_adam).
__global__ __launch_bounds__(256) void k_pack(Jobs<PackJob> q)
{
    const int jn = job_of(q);
    const PackJob a = q.j[jn];
    const int KC = a.cin_p / 16, NF = a.cout_p / 16;
    const long long e = ((long long)((int)blockIdx.x - q.first[jn]) * 256 + threadIdx.x) * 4;
    if (e >= a.total) return;
    float val[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (a.k32 == 2) {
        const int lane = (int)((e >> 3) & 63);
        const long long u = e >> 9;
        const int n = (int)(u % NF), t = 4 * (int)(u / NF) + (lane >> 4), co = 16 * n + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int j = (int)(e & 7) + r;
            if (t < 27 && j < a.cin && co < a.cout) val[r] = a.w[((long long)t * a.w_cin + j) * a.cout + co];
        }
    } else {
        const int sh = a.k32 ? 9 : 8;
        const int lane = (int)((e >> (sh - 6)) & 63), kc = a.k32 ? KC / 2 : KC;
        long long u = e >> sh;
        const int n = (int)(u % NF);
        u /= NF;
        const int c = (int)(u % kc), t = (int)(u / kc);
        const int k0 = a.k32 ? 32 * c + 8 * (lane >> 4) + (int)(e & 7) : 16 * c + 4 * (lane >> 4);   // input channels of this conv
        const int j = 16 * n + (lane & 15);              // output channel of this conv
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int k = k0 + r;
            if (!a.transpose) {
                if (k < a.cin && j < a.cout) val[r] = a.w[((long long)t * a.w_cin + k) * a.cout + j];
            } else {
                // adjoint: this conv maps cout-channel gradients to cin-channel ones
                const int tm = a.ntap - 1 - t;
                if (k < a.cout && j < a.cin) val[r] = a.w[((long long)tm * a.w_cin + j) * a.cout + k];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 4; r++) a.out[e + r] = f2bf(val[r]);
}

// ---------------------------------------------------------------- weight gradient
// Partial dW of one group of output tiles:
//   P[group][tap][ci][co] = sum_{v in the group's tiles} X[p(v, tap)][ci] dY[v][co]
// Both MFMA operands have the voxels along K while the tensors are
// channels-last, so the tiles are staged voxel-major (16-byte global-to-LDS
// copies, all in flight) and read back transposed: ds_read_b64_tr_b16 gives
// each lane four voxels of its channel (lane l of 16 addresses 8 bytes of
// voxel l / 4, and receives channel l of the four voxels).  The K positions of
// a step are any 32 voxels of the tile's (z, x) plane at one y, so a tile may
// have any shape; A and B use the same order.
//
// A workgroup takes one z tap, 16 ncf input channels and 16 NF nch output
// channels; its four waves split those (ncf x nch) and, where they do not
// fill four waves, the K steps (nkh).  A wave holds the NT x NT in-plane taps
// in registers: an input row r meets the gradient rows r - tb, so each A
// fragment feeds up to NT * NF MFMAs and the LDS reads (about 0.7 of the MFMA
// time at NF = 2) do not bound it.
// Measured on a training batch (8 boxes of 40 x 24 x 40, all 15 layers): 0.70 ms,
// 250 TFLOP/s; 4.4 ms before (channel-major LDS tiles filled by 2-byte stores,
// A fragments from eight 2-byte reads each).
typedef __attribute__((address_space(3))) s4 lds_s4;

// Eight K elements (two transposed reads) of one operand fragment; byte LDS offsets.
__device__ __forceinline__ b8 tr_frag(const char *sm, int lo, int hi)
{
    const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(sm + lo));
    const s4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(sm + hi));
    return __builtin_bit_cast(b8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int KIND, int NF>
__global__ __launch_bounds__(256, 3) void k_wgrad(WgradArgs a, WgradPlan p)
{
    constexpr int NT = KIND == KIND_C3 || KIND == KIND_UP ? 3 : (KIND == KIND_DOWN ? 2 : 1);
    constexpr int S = KIND == KIND_DOWN ? 2 : 1;
    constexpr int RY = S * (WTY - 1) + NT;
    typedef __attribute__((address_space(3))) void lds_void;
    typedef const __attribute__((address_space(1))) void glob_void;
    extern __shared__ uint4 smem[];
    char *sm = (char *)smem;
    int *tab = (int *)smem;            // per position: byte offset of its X row / 32 << 16 | column
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // the variants (z tap, channel blocks) of one group run on one XCD at about the same time (the
    // dispatcher deals workgroups to the eight XCDs in turn), sharing its tiles in that L2
    const int q8 = blockIdx.x >> 3;
    const int var = q8 % p.nvar, group = (q8 / p.nvar) * 8 + (blockIdx.x & 7);
    if (group >= p.groups) return;
    const int ta = var % NT, cb = (var / NT) % p.ncb, cg = var / (NT * p.ncb);
    const int cf = wv % p.ncf, ch = (wv / p.ncf) % p.nch, kh = wv / (p.ncf * p.nch);
    const int XP = 2 * p.ncf, GP = 2 * NF * p.nch;       // 16-byte pieces per voxel
    const int xrow = 16 * XP, grow = 16 * GP;            // bytes per voxel
    const int npos = 32 * p.ns, nreal = p.TZ * p.TX;
    const int ci0 = 16 * p.ncf * cb, co0 = 16 * NF * p.nch * cg;
    for (int e = tid; e < npos; e += 256) {
        const int z = div_by(e, p.mTX, p.TX), x = e - z * p.TX;
        tab[e] = e < nreal ? ((z * RY * p.HX * xrow) >> 5 << 16 | S * x) : 0;
    }
    f4 acc[NT][NT][NF];
#pragma unroll
    for (int tc = 0; tc < NT; tc++)
#pragma unroll
        for (int tb = 0; tb < NT; tb++)
#pragma unroll
            for (int n = 0; n < NF; n++) acc[tc][tb][n] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    const int g = lane >> 4, j = (lane & 15) >> 2, p8 = 8 * (lane & 3);
    // 32-byte channel chunks are swizzled so that the four voxels of a 16-lane group hit distinct banks
    const int gsw = GP == 8 ? j : (GP == 4 ? j >> 1 : 0);
    const int nx = p.TZ * RY * p.HX * XP, ng = WTY * npos * GP;
    const VoxelIndex xi(a.ih, a.iw, a.cx, p.wide), gi(a.oh, a.ow, a.cg, p.wide);
    const int tile_end = (int)min((long long)p.ntiles, (group + 1LL) * p.tpg);
    for (int tile = group * p.tpg; tile < tile_end; tile++) {
        int b = tile;
        const int x0 = (b % p.tiles_x) * p.TX;
        b /= p.tiles_x;
        const int y0 = (b % p.tiles_y) * WTY;
        b /= p.tiles_y;
        const int z0 = (b % p.tiles_z) * p.TZ, bn = b / p.tiles_z;
        const uint16_t *xb = a.x + (size_t)bn * a.id * a.ih * a.iw * a.cx + a.x_off + ci0;
        const uint16_t *gb = a.g + (size_t)bn * a.od * a.oh * a.ow * a.cg + a.g_off + co0;
        for (int s0 = 64 * wv; s0 < nx; s0 += 256) {
            const int s = s0 + lane;
            if (s >= nx) break;
            const int v = XP == 4 ? s >> 2 : s >> 1, ph = s & (XP - 1);
            const int q = div_by(v, p.mHX, p.HX), col = v - q * p.HX;
            const int z = q / RY, r = q - z * RY;
            const int c8 = 8 * (XP == 4 ? ph ^ (col & 2) : ph);
            int gz, gy, gx;
            bool in;
            if (KIND == KIND_UP) {
                gz = z0 + z + ta - 1; gy = y0 + r - 1; gx = x0 + col - 1;
                in = gz >= 0 && gy >= 0 && gx >= 0 && gz < 2 * a.id && gy < 2 * a.ih && gx < 2 * a.iw;
                gz >>= 1; gy >>= 1; gx >>= 1;
            } else {
                constexpr int P = KIND == KIND_C3 ? 1 : 0;
                gz = S * (z0 + z) + ta - P; gy = S * y0 + r - P; gx = S * x0 + col - P;
                in = gz >= 0 && gy >= 0 && gx >= 0 && gz < a.id && gy < a.ih && gx < a.iw;
            }
            in &= ci0 + c8 < a.cin;
            const uint16_t *src = in ? xb + xi(gz, gy, gx) + c8 : g_zero_piece;
            if (p.x16) __builtin_amdgcn_global_load_lds((glob_void *)src, (lds_void *)(sm + p.x_off + 16 * s0), 16, 0, 0);
            else *(uint4 *)(sm + p.x_off + 16 * s) = load_piece(src, 8);
        }
        for (int s0 = 64 * wv; s0 < ng; s0 += 256) {
            const int s = s0 + lane;
            const int v = GP == 8 ? s >> 3 : (GP == 4 ? s >> 2 : s >> 1), ph = s & (GP - 1);
            const int yo = div_by(v, p.mNP, npos), pos = v - yo * npos;
            const int z = div_by(pos, p.mTX, p.TX), x = pos - z * p.TX;
            const int c8 = 8 * (GP == 8 ? ph ^ ((pos & 3) << 1) : (GP == 4 ? ph ^ (pos & 2) : ph));
            const int gz = z0 + z, gy = y0 + yo, gx = x0 + x, left = a.cout - co0 - c8;
            const bool in = pos < nreal && gz < a.od && gy < a.oh && gx < a.ow && left > 0;
            const uint16_t *src = in ? gb + gi(gz, gy, gx) + c8 : g_zero_piece;
            if (p.g16) __builtin_amdgcn_global_load_lds((glob_void *)src, (lds_void *)(sm + p.g_off + 16 * s0), 16, 0, 0);
            else *(uint4 *)(sm + p.g_off + 16 * s) = load_piece(src, in ? min(left, 8) : 8);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the copies are not tracked by the compiler
        __syncthreads();
        for (int ks = kh; ks < p.ns; ks += p.nkh) {
            int ax[NT][2], ag[2];
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int pos = 32 * ks + 8 * g + 4 * h + j;
                const int e = tab[pos];
                const int row = p.x_off + (e >> 16 << 5);
#pragma unroll
                for (int tc = 0; tc < NT; tc++) {
                    const int col = (e & 0xffff) + tc;
                    ax[tc][h] = row + col * xrow + 32 * (XP == 4 ? cf ^ ((col >> 1) & 1) : 0) + p8;
                }
                ag[h] = p.g_off + pos * grow + p8;
            }
            b8 Bv[WTY][NF];
#pragma unroll
            for (int r = 0; r < RY; r++) {
                if (r % S == 0 && r / S < WTY)
#pragma unroll
                    for (int n = 0; n < NF; n++) {
                        const int o = r / S * npos * grow + 32 * ((ch * NF + n) ^ gsw);
                        Bv[r / S][n] = tr_frag(sm, ag[0] + o, ag[1] + o);
                    }
#pragma unroll
                for (int tc = 0; tc < NT; tc++) {
                    const int o = r * p.HX * xrow;
                    const b8 Av = tr_frag(sm, ax[tc][0] + o, ax[tc][1] + o);
#pragma unroll
                    for (int tb = 0; tb < NT; tb++) {
                        if (r < tb || (r - tb) % S || (r - tb) / S >= WTY) continue;
#pragma unroll
                        for (int n = 0; n < NF; n++)
                            acc[tc][tb][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Av, Bv[(r - tb) / S][n], acc[tc][tb][n], 0, 0, 0);
                    }
                }
            }
        }
        __syncthreads();
    }
    // waves that share their channels and split the K steps: sums added through LDS, one after the other
    constexpr int NA = NT * NT * NF;
    f4 *red = (f4 *)sm + (wv % (p.ncf * p.nch)) * NA * 64 + lane;
    for (int k = 1; k < p.nkh; k++) {
        if (kh == k)
#pragma unroll
            for (int i = 0; i < NA; i++) red[64 * i] = acc[i / (NT * NF)][(i / NF) % NT][i % NF];
        __syncthreads();
        if (kh == 0)
#pragma unroll
            for (int i = 0; i < NA; i++) acc[i / (NT * NF)][(i / NF) % NT][i % NF] += red[64 * i];
        __syncthreads();
    }
    if (kh != 0) return;
    // D[i][j]: ci = 4 (lane / 16) + r, co = lane % 16 of the wave's fragments
    const int ci = ci0 + 16 * cf + 4 * g;
    if (ci >= a.cin) return;
#pragma unroll
    for (int tc = 0; tc < NT; tc++)
#pragma unroll
        for (int tb = 0; tb < NT; tb++) {
            float *P = a.partial + (((long long)group * NT * NT * NT + (ta * NT + tb) * NT + tc) * a.cin + ci) * a.cout;
#pragma unroll
            for (int n = 0; n < NF; n++) {
                const int co = co0 + 16 * (ch * NF + n) + (lane & 15);
                if (co >= a.cout) continue;
#pragma unroll
                for (int r = 0; r < 4; r++) P[(long long)r * a.cout + co] = acc[tc][tb][n][r];
            }
        }
}

// Sum of the partials: a workgroup takes 64 V outputs, its NW waves every NW-th
// partial (eight loads in flight), added through LDS.  One thread per output
// over all partials left the card idle: 38 us a layer on a training batch.
template <int V, int NW>
__global__ __launch_bounds__(64 * NW) void k_reduce_partials(const float *partial, int nchunk, long long per, float *out,
                                                             int accumulate)
{
    __shared__ float red[NW][64 * V];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long long e = ((long long)blockIdx.x * 64 + lane) * V;
    const bool in = e < per;
    float s[V] = {};
    if (in) {
        int c = w;
        for (; c + 7 * NW < nchunk; c += 8 * NW) {
            float t[8][V];
#pragma unroll
            for (int u = 0; u < 8; u++)
#pragma unroll
                for (int k = 0; k < V; k++) t[u][k] = partial[(long long)(c + u * NW) * per + e + k];
#pragma unroll
            for (int u = 0; u < 8; u++)
#pragma unroll
                for (int k = 0; k < V; k++) s[k] += t[u][k];
        }
        for (; c < nchunk; c += NW)
#pragma unroll
            for (int k = 0; k < V; k++) s[k] += partial[(long long)c * per + e + k];
    }
#pragma unroll
    for (int k = 0; k < V; k++) red[w][lane * V + k] = s[k];
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * V; i += 64 * NW) {
        const long long o = (long long)blockIdx.x * 64 * V + i;
        if (o >= per) continue;
        float t = accumulate ? out[o] : 0.0f;
#pragma unroll
        for (int k = 0; k < NW; k++) t += red[k][i];
        out[o] = t;
    }
}

// bias gradient: gb[co] (+)= sum over voxels of dY[v][co].  Each workgroup
// sums a chunk of voxels for every channel (consecutive threads read
// consecutive channels of a voxel), reduces in LDS and adds its partial sums
// with one float atomic per channel; gb is cleared first unless accumulating.
// The voxels are cut into about 512 chunks, two workgroups per CU (at 8,192
// voxels a chunk the largest layer of a training batch had 38 workgroups and
// took 80 us), of eight voxels a lane at least and 300 at most up to 16 channels,
// whose atomics show (4 channels, 200,000 voxels: 12.5 us in 512 chunks, 7.6 in
// 98), and of multiples of 256 voxels, which start on whole cache lines (16
// channels, 2.5 million voxels: 20.0 -> 18.4 us; 64 and 200,000: 17.2 -> 14.2).

__global__ void k_fill_f(float *p, int n, float v)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ __launch_bounds__(256) void k_bias_grad(const uint16_t *g, long long nvox, int cg, int g_off, int cout,
                                                   float *gb, int chunk)
{
    __shared__ float red[256];
    const int vl = 256 / cout;                       // voxel lanes (cout <= 128)
    const int co = threadIdx.x % cout, lv = threadIdx.x / cout;
    const long long v0 = (long long)blockIdx.x * chunk, v1 = min(nvox, v0 + chunk);
    float sum = 0.0f;
    if (lv < vl)
        for (long long v = v0 + lv; v < v1; v += vl) sum += bf2f(g[v * cg + g_off + co]);
    red[threadIdx.x] = lv < vl ? sum : 0.0f;
    __syncthreads();
    if (threadIdx.x < cout) {
        float t = 0.0f;
        for (int k = 0; k < vl; k++) t += red[k * cout + threadIdx.x];
        atomicAdd(gb + threadIdx.x, t);
    }
}

// The same sum with 4 channels per thread (8-byte loads) and four voxels in
// flight per thread; needs cout, cg and g_off multiples of 4.
__global__ __launch_bounds__(256) void k_bias_grad4(const uint16_t *g, long long nvox, int cg, int g_off, int cout,
                                                    float *gb, int chunk)
{
    __shared__ float red[256 * 4];
    const int cq = cout / 4;                         // threads per voxel
    const int vl = 256 / cq;                         // voxel lanes
    const int q = threadIdx.x % cq, lv = threadIdx.x / cq;
    const long long v0 = (long long)blockIdx.x * chunk, v1 = min(nvox, v0 + chunk);
    float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (lv < vl) {
        const uint16_t *gp = g + g_off + 4 * q;
        long long v = v0 + lv;
        for (; v + 3 * vl < v1; v += 4 * vl) {
            uint2 r[4];
#pragma unroll
            for (int u = 0; u < 4; u++) r[u] = *(const uint2 *)(gp + (v + u * vl) * cg);
#pragma unroll
            for (int u = 0; u < 4; u++) {
                sum[0] += __uint_as_float(r[u].x << 16);
                sum[1] += __uint_as_float(r[u].x & 0xffff0000u);
                sum[2] += __uint_as_float(r[u].y << 16);
                sum[3] += __uint_as_float(r[u].y & 0xffff0000u);
            }
        }
        for (; v < v1; v += vl) {
            const uint2 r = *(const uint2 *)(gp + v * cg);
            sum[0] += __uint_as_float(r.x << 16);
            sum[1] += __uint_as_float(r.x & 0xffff0000u);
            sum[2] += __uint_as_float(r.y << 16);
            sum[3] += __uint_as_float(r.y & 0xffff0000u);
        }
    }
#pragma unroll
    for (int k = 0; k < 4; k++) red[k * 256 + threadIdx.x] = lv < vl ? sum[k] : 0.0f;
    __syncthreads();
    if (threadIdx.x < cout) {
        const int co = threadIdx.x, qq = co / 4, k = co % 4;
        float t = 0.0f;
        for (int l = 0; l < vl; l++) t += red[k * 256 + l * cq + qq];
        atomicAdd(gb + co, t);
    }
}

// ---------------------------------------------------------------- elementwise and resampling
// g <- g * (y > 0) over a channel slice (ReLU backward; y is the layer output)
__global__ void k_relu_bwd(uint16_t *g, int cg, int g_off, const uint16_t *y, int cy, int y_off, long long nvox, int c)
{
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < nvox * c; e += (long long)gridDim.x * blockDim.x) {
        long long v = e / c;
        int ch = (int)(e % c);
        if (!(bf2f(y[v * cy + y_off + ch]) > 0.0f)) g[v * cg + g_off + ch] = 0;
    }
}

// The same with 8 channels per thread (16-byte loads and stores; c = 8 << cs): one
// channel per thread spent its time on the index divisions.
__global__ __launch_bounds__(256) void k_relu_bwd8(uint16_t *g, int cg, int g_off, const uint16_t *y, int cy, int y_off,
                                                   long long n, int cs)
{
    for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
        const long long v = e >> cs;
        const int c = 8 * (int)(e & ((1 << cs) - 1));
        uint4 *gp = (uint4 *)(g + v * cg + g_off + c);
        const uint4 yv = *(const uint4 *)(y + v * cy + y_off + c);
        uint4 gv = *gp;
        auto keep = [](uint32_t gw, uint32_t yw) {
            return (bf2f((uint16_t)yw) > 0.0f ? gw & 0xffffu : 0u) | (bf2f((uint16_t)(yw >> 16)) > 0.0f ? gw & 0xffff0000u : 0u);
        };
        gv.x = keep(gv.x, yv.x);
        gv.y = keep(gv.y, yv.y);
        gv.z = keep(gv.z, yv.z);
        gv.w = keep(gv.w, yv.w);
        *gp = gv;
    }
}

// coarse[U] = sum of the 8 fine children (nearest-upsampling backward)
__global__ void k_up_bwd(const uint16_t *fine, int cf, int f_off, uint16_t *coarse, int cc, int c_off, int n, int d, int h,
                         int w, int c)
{
    const long long total = (long long)n * d * h * w * c;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total; e += (long long)gridDim.x * blockDim.x) {
        int ch = (int)(e % c);
        long long v = e / c;
        int x = (int)(v % w);
        long long q = v / w;
        int y = (int)(q % h);
        q /= h;
        int z = (int)(q % d);
        int nn = (int)(q / d);
        float s = 0.0f;
        for (int a = 0; a < 2; a++)
            for (int b = 0; b < 2; b++)
                for (int cc2 = 0; cc2 < 2; cc2++) {
                    long long fv = (((long long)nn * 2 * d + 2 * z + a) * 2 * h + 2 * y + b) * 2 * w + 2 * x + cc2;
                    s += bf2f(fine[fv * cf + f_off + ch]);
                }
        coarse[v * cc + c_off + ch] = f2bf(s);
    }
}

// The same with 8 channels per thread (c = 8 << cs).
__global__ __launch_bounds__(256) void k_up_bwd8(const uint16_t *fine, int cf, int f_off, uint16_t *coarse, int cc, int c_off,
                                                 int n, int d, int h, int w, int cs)
{
    const long long total = ((long long)n * d * h * w) << cs;
    for (long long e = blockIdx.x * 256LL + threadIdx.x; e < total; e += (long long)gridDim.x * 256) {
        const int ch = 8 * (int)(e & ((1 << cs) - 1));
        const long long v = e >> cs;
        const int x = (int)(v % w);
        long long q = v / w;
        const int y = (int)(q % h);
        q /= h;
        const int z = (int)(q % d), nn = (int)(q / d);
        const uint16_t *f = fine + ((((long long)nn * 2 * d + 2 * z) * 2 * h + 2 * y) * 2 * w + 2 * x) * cf + f_off + ch;
        uint4 r[8];
#pragma unroll
        for (int k = 0; k < 8; k++)
            r[k] = *(const uint4 *)(f + (((long long)(k >> 2) * 2 * h + ((k >> 1) & 1)) * 2 * w + (k & 1)) * cf);
        float s[8] = {};
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const uint32_t u[4] = {r[k].x, r[k].y, r[k].z, r[k].w};
#pragma unroll
            for (int j = 0; j < 4; j++) {
                s[2 * j] += __uint_as_float(u[j] << 16);
                s[2 * j + 1] += __uint_as_float(u[j] & 0xffff0000u);
            }
        }
        *(uint4 *)(coarse + v * cc + c_off + ch) = make_uint4(f2bf2(s[0], s[1]), f2bf2(s[2], s[3]), f2bf2(s[4], s[5]), f2bf2(s[6], s[7]));
    }
}

// dX of the 2^3 stride-2 convolution: dX[u] = dY[u / 2] W[u % 2]^T (weights
// rounded to BF16 like those of every other adjoint, FP32 accumulation)
__global__ void k_down_dgrad(const uint16_t *g, int cg, int g_off, const float *w, int cin, int cout, uint16_t *gx,
                             int cx, int x_off, int n, int d, int h, int wd, int accumulate)
{
    // (d, h, wd) are the fine sizes
    const long long total = (long long)n * d * h * wd * cin;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total; e += (long long)gridDim.x * blockDim.x) {
        int ci = (int)(e % cin);
        long long v = e / cin;
        int x = (int)(v % wd);
        long long q = v / wd;
        int y = (int)(q % h);
        q /= h;
        int z = (int)(q % d);
        int nn = (int)(q / d);
        int t = ((z & 1) * 2 + (y & 1)) * 2 + (x & 1);
        long long cv = (((long long)nn * (d / 2) + z / 2) * (h / 2) + y / 2) * (wd / 2) + x / 2;
        const float *wt = w + ((long long)t * cin + ci) * cout;
        float s = 0.0f;
        for (int co = 0; co < cout; co++) s += bf2f(g[cv * cg + g_off + co]) * bf2f(f2bf(wt[co]));
        if (accumulate) s += bf2f(gx[v * cx + x_off + ci]);
        gx[v * cx + x_off + ci] = f2bf(s);
    }
}

// The same adjoint on MFMA: for each of the 8 taps t it is a GEMM
//   D[ci][coarse voxel V] = sum_co W[t][ci][co] dY[V][co]
// whose result lands on the fine voxel 2 V + t.  A wave owns one tap
// (blockIdx.y), 16 MF coarse voxels and 16 NF input channels; the FP32 weights
// are the row operand, rounded to BF16 as they are read, so that a lane ends
// with four channels of one voxel (8-byte stores).  One wave over all eight
// taps with 2-byte stores kept too few bytes in flight: 245 and 137 us on the
// two stride-2 layers of a training batch.
template <int MF, int NF>
__global__ __launch_bounds__(256) void k_down_dgrad_mfma(const uint16_t *g, int cg, int g_off, const float *w, int cin,
                                                         int cout, uint16_t *gx, int cx, int x_off, int n, int d, int h,
                                                         int wd, int accumulate, int ncb)
{
    const int lane = threadIdx.x & 63, i = lane & 15, gq = lane >> 4;
    const int D2 = d / 2, H2 = h / 2, W2 = wd / 2;
    const int nvc = n * D2 * H2 * W2, t = blockIdx.y;
    const int wave = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int cb = wave % ncb * 16 * NF, V0 = wave / ncb * (16 * MF);
    if (V0 >= nvc) return;
    const int kc = cout / 16;
    const uint16_t *gp[MF];
#pragma unroll
    for (int f = 0; f < MF; f++) gp[f] = g + (long long)min(V0 + 16 * f + i, nvc - 1) * cg + g_off + 4 * gq;
    const float *wp = w + ((long long)t * cin + cb + i) * cout + 4 * gq;
    f4 acc[MF][NF];
#pragma unroll
    for (int f = 0; f < MF; f++)
#pragma unroll
        for (int nf = 0; nf < NF; nf++) acc[f][nf] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    for (int c = 0; c < kc; c++) {
        s4 A[MF];
#pragma unroll
        for (int f = 0; f < MF; f++) A[f] = __builtin_bit_cast(s4, *(const uint2 *)(gp[f] + 16 * c));
#pragma unroll
        for (int nf = 0; nf < NF; nf++) {
            const float4 wv = *(const float4 *)(wp + (long long)nf * 16 * cout + 16 * c);
            const s4 Bv = __builtin_bit_cast(s4, make_uint2(f2bf2(wv.x, wv.y), f2bf2(wv.z, wv.w)));
#pragma unroll
            for (int f = 0; f < MF; f++) acc[f][nf] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(Bv, A[f], acc[f][nf], 0, 0, 0);
        }
    }
    const bool x8 = cx % 4 == 0 && x_off % 4 == 0 && ((uintptr_t)gx & 7) == 0;
#pragma unroll
    for (int f = 0; f < MF; f++) {
        const int V = V0 + 16 * f + i;
        if (V >= nvc) continue;
        const int x = V % W2, y = (V / W2) % H2, z = (V / (W2 * H2)) % D2, nn = V / (W2 * H2 * D2);
        const long long fine = ((long long)(nn * d + 2 * z + (t >> 2)) * h + 2 * y + ((t >> 1) & 1)) * wd + 2 * x + (t & 1);
        uint16_t *op = gx + fine * cx + x_off + cb + 4 * gq;
#pragma unroll
        for (int nf = 0; nf < NF; nf++) {
            float val[4];
            uint16_t *o = op + 16 * nf;
            if (x8) {
                const uint2 old = accumulate ? *(const uint2 *)o : make_uint2(0u, 0u);
#pragma unroll
                for (int r = 0; r < 4; r++) val[r] = acc[f][nf][r];
                if (accumulate) {
                    val[0] += __uint_as_float(old.x << 16);
                    val[1] += __uint_as_float(old.x & 0xffff0000u);
                    val[2] += __uint_as_float(old.y << 16);
                    val[3] += __uint_as_float(old.y & 0xffff0000u);
                }
                *(uint2 *)o = make_uint2(f2bf2(val[0], val[1]), f2bf2(val[2], val[3]));
            } else {
#pragma unroll
                for (int r = 0; r < 4; r++) o[r] = f2bf(accumulate ? acc[f][nf][r] + bf2f(o[r]) : acc[f][nf][r]);
            }
        }
    }
}

// FP32 -> BF16 channel-slice copy (network input)
__global__ void k_to_bf16(const float *x, int cs, long long nvox, int c, uint16_t *y, int cy, int y_off, int c_pad)
{
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < nvox * c_pad; e += (long long)gridDim.x * blockDim.x) {
        long long v = e / c_pad;
        int ch = (int)(e % c_pad);
        y[v * cy + y_off + ch] = ch < c ? f2bf(x[v * cs + ch]) : (uint16_t)0;
    }
}

// The same with 8 channels per thread (c_pad = 8 << ps; x4: rows of whole float4).
__global__ __launch_bounds__(256) void k_to_bf16_8(const float *x, int cs, long long n, int c, uint16_t *y, int cy, int y_off,
                                                   int ps, int x4)
{
    for (long long e = blockIdx.x * 256LL + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
        const long long v = e >> ps;
        const int c0 = 8 * (int)(e & ((1 << ps) - 1));
        const float *xp = x + v * cs + c0;
        float f[8] = {};
        if (x4 && c0 + 8 <= c) {
            const float4 a = *(const float4 *)xp, b = *(const float4 *)(xp + 4);
            f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
            f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
        } else {
#pragma unroll
            for (int k = 0; k < 8; k++)
                if (c0 + k < c) f[k] = xp[k];
        }
        *(uint4 *)(y + v * cy + y_off + c0) = make_uint4(f2bf2(f[0], f[1]), f2bf2(f[2], f[3]), f2bf2(f[4], f[5]), f2bf2(f[6], f[7]));
    }
}

// Number of masked voxels (mask != 0): integer partial counts per workgroup
// added into the count slot (held as an int while counting), then turned
// into a float (exact below 2^24 voxels).
__global__ void k_mask_count(const float *mask, long long nvox, int *count)
{
    __shared__ int red[256];
    int c = 0;
    for (long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x; v < nvox; v += (long long)gridDim.x * blockDim.x)
        c += mask[v] != 0.0f;
    red[threadIdx.x] = c;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0 && red[0]) atomicAdd(count, red[0]);
}

__global__ void k_int_slot(int *slot, int to_float)
{
    if (to_float) *(float *)slot = (float)*slot;
    else *slot = 0;
}

// Masked mean-squared error and its gradient (BF16):
// loss_parts[block] = partial sums of mask (pred - target)^2, g = 2 (pred - target) / (count c)
// on masked voxels, 0 elsewhere (all cg channels written).
__global__ void k_masked_mse(const float *pred, int cp, const float *target, const float *mask, long long nvox, int c,
                             const float *count, uint16_t *g, int cg, float *loss_parts)
{
    __shared__ float red[256];
    const float cnt = (float)*(const int *)count * (float)c;
    const float inv_count = cnt > 0.0f ? 1.0f / cnt : 0.0f;
    float s = 0.0f;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < nvox * cg; e += (long long)gridDim.x * blockDim.x) {
        long long v = e / cg;
        int ch = (int)(e % cg);
        float gv = 0.0f;
        if (ch < c && mask[v] != 0.0f) {
            float d = pred[v * cp + ch] - target[v * c + ch];
            s += d * d;
            gv = 2.0f * d * inv_count;
        }
        g[e] = f2bf(gv);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss_parts[blockIdx.x] = red[0];
}

// Adam on FP32 master parameters (bias-corrected with step t)
// 1,024 elements per workgroup, 28 bytes each; every parameter tensor of the
// network in one launch (30 launches of a few microseconds each, with as many
// for the weight fragments, were 553 us an update; two are 61).
__global__ __launch_bounds__(256) void k_adam(Jobs<AdamJob> q, float lr, float b1, float b2, float eps, int t)
{
    const int jn = job_of(q);
    const AdamJob a = q.j[jn];
    const float c1 = 1.0f / (1.0f - powf(b1, (float)t)), c2 = 1.0f / (1.0f - powf(b2, (float)t));
    const long long base = (long long)((int)blockIdx.x - q.first[jn]) * 1024;
    auto update = [&](float &p, float g, float &m, float &v) {
        m = b1 * m + (1.0f - b1) * g;
        v = b2 * v + (1.0f - b2) * g * g;
        p -= lr * (m * c1) / (sqrtf(v * c2) + eps);
    };
    if (a.vec && base + 1024 <= a.n) {
        const long long e = base / 4 + threadIdx.x;
        const float4 g = ((const float4 *)a.g)[e];
        float4 p = ((float4 *)a.p)[e], m = ((float4 *)a.m)[e], v = ((float4 *)a.v)[e];
        update(p.x, g.x, m.x, v.x);
        update(p.y, g.y, m.y, v.y);
        update(p.z, g.z, m.z, v.z);
        update(p.w, g.w, m.w, v.w);
        ((float4 *)a.m)[e] = m;
        ((float4 *)a.v)[e] = v;
        ((float4 *)a.p)[e] = p;
        return;
    }
    for (long long e = base + threadIdx.x; e < a.n && e < base + 1024; e += 256) {
        float p = a.p[e], m = a.m[e], v = a.v[e];
        update(p, a.g[e], m, v);
        a.m[e] = m;
        a.v[e] = v;
        a.p[e] = p;
    }
}

// ---------------------------------------------------------------- crops of dense per-scene grids
// Bounding box of the nodes whose channel 0 is positive, one workgroup per
// grid: bbox[g] = (lo_x, lo_y, lo_z, hi_x, hi_y, hi_z), hi exclusive; an
// empty grid gives (0, 0, 0, 0, 0, 0).
__global__ __launch_bounds__(256) void k_bbox(const float *field, int cf, int R, int *bbox)
{
    __shared__ int red[6][256];
    const long long R3 = (long long)R * R * R;
    const float *f = field + (long long)blockIdx.x * R3 * cf;
    int lo[3] = {R, R, R}, hi[3] = {-1, -1, -1};
    for (long long c = threadIdx.x; c < R3; c += 256) {
        if (!(f[c * cf] > 0.0f)) continue;
        const int ii[3] = {(int)(c / ((long long)R * R)), (int)((c / R) % R), (int)(c % R)};
        for (int d = 0; d < 3; d++) {
            lo[d] = min(lo[d], ii[d]);
            hi[d] = max(hi[d], ii[d]);
        }
    }
    for (int d = 0; d < 3; d++) {
        red[d][threadIdx.x] = lo[d];
        red[3 + d][threadIdx.x] = hi[d];
    }
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o)
            for (int d = 0; d < 3; d++) {
                red[d][threadIdx.x] = min(red[d][threadIdx.x], red[d][threadIdx.x + o]);
                red[3 + d][threadIdx.x] = max(red[3 + d][threadIdx.x], red[3 + d][threadIdx.x + o]);
            }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const bool empty = red[3][0] < 0;
        for (int d = 0; d < 3; d++) {
            bbox[6 * blockIdx.x + d] = empty ? 0 : red[d][0];
            bbox[6 * blockIdx.x + 3 + d] = empty ? 0 : red[3 + d][0] + 1;
        }
    }
}

// Crop origin per grid: the box of size (D, H, W) centred on bbox, moved
// inside [0, R).
__global__ void k_crop_origin(const int *bbox, int n, int R, int D, int H, int W, int *origin)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    const int size[3] = {D, H, W};
    for (int d = 0; d < 3; d++) {
        const int lo = bbox[6 * g + d], hi = bbox[6 * g + 3 + d];
        int o = (lo + hi - size[d]) / 2;
        o = max(0, min(o, R - size[d]));
        origin[3 * g + d] = o;
    }
}

// dst[g][z][y][x][:c] = src[g][oz + z][oy + y][ox + x][:c]  (crop), or the
// reverse with zeros outside the crop (uncrop: dst is the full grid).
__global__ void k_crop(const float *src, int c, int n, int R, const int *origin, int D, int H, int W, float *dst,
                       int uncrop)
{
    const long long R3 = (long long)R * R * R;
    const long long per = uncrop ? R3 : (long long)D * H * W;
    const long long total = per * n * c;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total; e += (long long)gridDim.x * blockDim.x) {
        const int ch = (int)(e % c);
        const long long v = e / c;
        const int g = (int)(v / per);
        const long long l = v - (long long)g * per;
        const int* o = origin + 3 * g;
        if (!uncrop) {
            const int z = (int)(l / ((long long)H * W)), y = (int)((l / W) % H), x = (int)(l % W);
            const long long sv = (((long long)g * R + o[0] + z) * R + o[1] + y) * R + o[2] + x;
            dst[e] = src[sv * c + ch];
        } else {
            const int i = (int)(l / ((long long)R * R)), j = (int)((l / R) % R), k = (int)(l % R);
            const int z = i - o[0], y = j - o[1], x = k - o[2];
            float val = 0.0f;
            if (z >= 0 && y >= 0 && x >= 0 && z < D && y < H && x < W)
                val = src[((((long long)g * D + z) * H + y) * W + x) * c + ch];
            dst[e] = val;
        }
    }
}

// ---------------------------------------------------------------- launchers
static unsigned grid_for(long long n, int per = 256)
{
    long long b = (n + per - 1) / per;
    return (unsigned)(b < 16384 ? (b < 1 ? 1 : b) : 16384);
}

template <int NF, int KIND>
static hipError_t conv_pos(const ConvArgs &a, hipStream_t st)
{
    ConvPlan p{};
    int FR = 0;
    if (!conv_plan(a, NF, p, FR)) return hipErrorInvalidValue;
    const unsigned g = (unsigned)((p.ntiles + 7) / 8 * 8 * p.nco), t = 64 * p.PW * p.CW;
    const void *fn = FR == 8 ? (const void *)k_conv_pos<NF, KIND, 8> : (FR == 6 ? (const void *)k_conv_pos<NF, KIND, 6> : (const void *)k_conv_pos<NF, KIND, 4>);
    ConvArgs args = a;
    void *params[] = {&args, &p};
    return hipLaunchKernel(fn, dim3(g), dim3(t), params, p.lds, st);
}

template <int KIND>
static hipError_t conv_lds(const ConvArgs &a, hipStream_t st)
{
    const int nf = (a.cout + 15) / 16;
    if (a.cin % 32 == 0)   // the weights were packed as 16x16x32 fragments (same condition in pack)
        return nf == 1 ? conv_pos<1, KIND>(a, st) : conv_pos<2, KIND>(a, st);
    const long long tiles = (long long)a.n * ((a.od + TLZ - 1) / TLZ) * ((a.oh + TLY - 1) / TLY) * ((a.ow + TLX - 1) / TLX);
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    const unsigned g = (unsigned)tiles;
    switch (nf) {
    case 1: k_conv_lds<1, KIND><<<g, 256, 0, st>>>(a); break;
    case 2: k_conv_lds<2, KIND><<<g, 256, 0, st>>>(a); break;
    case 4: k_conv_lds<4, KIND><<<g, 256, 0, st>>>(a); break;
    case 8: k_conv_lds<8, KIND><<<g, 256, 0, st>>>(a); break;
    }
    return hipGetLastError();
}

template <int NF, int KC>
static hipError_t conv_direct_kc(const ConvArgs &a, hipStream_t st)
{
    const long long nvox = (long long)a.n * a.od * a.oh * a.ow;
    const int ncg = (a.cout + 16 * NF - 1) / (16 * NF);
    // voxels per wave: 64, or fewer while the launch has less than 32 waves per CU
    int mf = 4;
    while (mf > 1 && (nvox + 16 * mf - 1) / (16 * mf) * ncg < 8192) mf /= 2;
    const long long wgs = ((nvox + 16 * mf - 1) / (16 * mf) * ncg + 3) / 4;
    if (wgs > 0x7fffffff) return hipErrorInvalidValue;
    const unsigned g = (unsigned)wgs;
    if (mf == 4) k_conv<4, NF, KC><<<g, 256, 0, st>>>(a, ncg);
    else if (mf == 2) k_conv<2, NF, KC><<<g, 256, 0, st>>>(a, ncg);
    else k_conv<1, NF, KC><<<g, 256, 0, st>>>(a, ncg);
    return hipGetLastError();
}

template <int NF>
static hipError_t conv_direct(const ConvArgs &a, hipStream_t st)
{
    if (a.cin == 32) return conv_direct_kc<NF, 2>(a, st);
    if (a.cin == 64) return conv_direct_kc<NF, 4>(a, st);
    return conv_direct_kc<NF, 0>(a, st);
}

hipError_t conv(const ConvArgs &a, hipStream_t st)
{
    const int nf = (a.cout + 15) / 16;
    if (nf != 1 && nf != 2 && nf != 4 && nf != 8) return hipErrorInvalidValue;
    if (a.kind == KIND_C3 && a.cin == 8) {
        ConvPlan p{};
        if (a.cx % 8 || a.x_off % 8 || ((uintptr_t)a.x & 15) || !first_plan(a, p)) return hipErrorInvalidValue;
        const unsigned g = (unsigned)((p.ntiles + 7) / 8 * 8);
        switch (nf) {
        case 1: k_conv_first<1><<<g, 256, p.lds, st>>>(a, p); break;
        case 2: k_conv_first<2><<<g, 256, p.lds, st>>>(a, p); break;
        case 4: k_conv_first<4><<<g, 256, p.lds, st>>>(a, p); break;
        case 8: k_conv_first<8><<<g, 256, p.lds, st>>>(a, p); break;
        }
        return hipGetLastError();
    }
    if (a.kind == KIND_C3) return conv_lds<KIND_C3>(a, st);
    if (a.kind == KIND_UP) return conv_lds<KIND_UP>(a, st);
    if (nf == 1) return conv_direct<1>(a, st);
    // 64 channels per wave read each input line once for them; on small grids 32, for more waves
    const long long nvox = (long long)a.n * a.od * a.oh * a.ow;
    return nf >= 4 && (nvox + 15) / 16 * (nf / 4) >= 2048 ? conv_direct<4>(a, st) : conv_direct<2>(a, st);
}

PackJob pack_job(const float *w, int ntap, int w_cin, int cin, int cout, int cin_p, int cout_p, int transpose, uint16_t *out)
{
    // 3^3 kernels with a multiple of 32 input channels run on 16x16x32 fragments, and so does the
    // 3^3 layer over 8 input channels (taps folded into K)
    const int k32 = ntap == 27 && !transpose && cin == 8 ? 2 : (ntap == 27 && cin_p % 32 == 0);
    const long long total = k32 == 2 ? (long long)FIRST_STEPS * (cout_p / 16) * 512
                                     : (long long)ntap * (cin_p / 16) * (cout_p / 16) * 256;
    return {w, out, total, ntap, w_cin, cin, cout, cin_p, cout_p, transpose, k32};
}

// One launch of `count` jobs (Jobs::MAX at most); size(job): its workgroups.
template <class Job, class Size, class Launch>
static hipError_t launch_jobs(const Job *jobs, int count, Size size, Launch launch)
{
    if (count > Jobs<Job>::MAX) return hipErrorInvalidValue;
    Jobs<Job> q;
    q.count = count;
    q.first[0] = 0;
    for (int j = 0; j < count; j++) {
        q.j[j] = jobs[j];
        q.first[j + 1] = q.first[j] + size(jobs[j]);
    }
    launch(q, (unsigned)q.first[count]);
    return hipGetLastError();
}

hipError_t pack(const PackJob *jobs, int count, hipStream_t st)
{
    return launch_jobs(jobs, count, [](const PackJob &j) { return (int)((j.total + 1023) / 1024); },
                       [&](const Jobs<PackJob> &q, unsigned g) { k_pack<<<g, 256, 0, st>>>(q); });
}

static hipError_t reduce_partials(const float *partial, int n, long long per, float *out, int accumulate, hipStream_t st)
{
    const bool v4 = per % 4 == 0 && ((uintptr_t)partial & 15) == 0;
    const long long w = v4 ? 256 : 64, wgs = (per + w - 1) / w;
    if (wgs > 0x7fffffff) return hipErrorInvalidValue;
    const unsigned g = (unsigned)wgs;
    if (v4 && n >= 64) k_reduce_partials<4, 16><<<g, 1024, 0, st>>>(partial, n, per, out, accumulate);
    else if (v4) k_reduce_partials<4, 4><<<g, 256, 0, st>>>(partial, n, per, out, accumulate);
    else k_reduce_partials<1, 4><<<g, 256, 0, st>>>(partial, n, per, out, accumulate);
    return hipGetLastError();
}

template <int KIND>
static hipError_t wgrad_kind(const WgradArgs &a, hipStream_t st)
{
    WgradPlan p{};
    if (!wgrad_plan(a, p)) return hipErrorInvalidValue;
    const unsigned g = (unsigned)((p.groups + 7) / 8 * 8 * p.nvar);
    if ((a.cout + 15) / 16 >= 2) k_wgrad<KIND, 2><<<g, 256, p.lds, st>>>(a, p);
    else k_wgrad<KIND, 1><<<g, 256, p.lds, st>>>(a, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int nt = KIND == KIND_C3 || KIND == KIND_UP ? 27 : (KIND == KIND_DOWN ? 8 : 1);
    return reduce_partials(a.partial, p.groups, (long long)nt * a.cin * a.cout, a.gw, a.accumulate, st);
}

hipError_t wgrad(const WgradArgs &a, hipStream_t st)
{
    if (a.kind == KIND_C3) return wgrad_kind<KIND_C3>(a, st);
    if (a.kind == KIND_UP) return wgrad_kind<KIND_UP>(a, st);
    if (a.kind == KIND_DOWN) return wgrad_kind<KIND_DOWN>(a, st);
    return wgrad_kind<KIND_C1>(a, st);
}

hipError_t bias_grad(const uint16_t *g, long long nvox, int cg, int g_off, int cout, float *gb, int accumulate,
                     hipStream_t st)
{
    if (cout > 128) return hipErrorInvalidValue;
    if (!accumulate) k_fill_f<<<(cout + 63) / 64, 64, 0, st>>>(gb, cout, 0.0f);
    const bool v4 = cout % 4 == 0 && cg % 4 == 0 && g_off % 4 == 0 && ((uintptr_t)g & 7) == 0;
    const long long lanes = v4 ? 256 / (cout / 4) : 256 / cout;   // voxels that a workgroup reads at once
    const int most = v4 && cout <= 16 ? 304 : 512;
    const long long chunk = std::min((std::max(8 * lanes, (nvox + most - 1) / most) + 255) & ~255LL, 1LL << 20);
    const long long nb = (nvox + chunk - 1) / chunk;
    if (v4)
        k_bias_grad4<<<(unsigned)nb, 256, 0, st>>>(g, nvox, cg, g_off, cout, gb, (int)chunk);
    else
        k_bias_grad<<<(unsigned)nb, 256, 0, st>>>(g, nvox, cg, g_off, cout, gb, (int)chunk);
    return hipGetLastError();
}

// log2(c / 8) when c is 8 times a power of two, else -1.
static int vec8(int c)
{
    for (int s = 0; s < 8; s++)
        if (c == 8 << s) return s;
    return -1;
}

hipError_t relu_bwd(uint16_t *g, int cg, int g_off, const uint16_t *y, int cy, int y_off, long long nvox, int c,
                    hipStream_t st)
{
    const int cs = vec8(c);
    if (cs >= 0 && cg % 8 == 0 && g_off % 8 == 0 && cy % 8 == 0 && y_off % 8 == 0 && !(((uintptr_t)g | (uintptr_t)y) & 15)) {
        k_relu_bwd8<<<grid_for(nvox << cs), 256, 0, st>>>(g, cg, g_off, y, cy, y_off, nvox << cs, cs);
        return hipGetLastError();
    }
    k_relu_bwd<<<grid_for(nvox * c), 256, 0, st>>>(g, cg, g_off, y, cy, y_off, nvox, c);
    return hipGetLastError();
}

hipError_t up_bwd(const uint16_t *fine, int cf, int f_off, uint16_t *coarse, int cc, int c_off, int n, int d, int h, int w,
                  int c, hipStream_t st)
{
    const int cs = vec8(c);
    if (cs >= 0 && cf % 8 == 0 && f_off % 8 == 0 && cc % 8 == 0 && c_off % 8 == 0 && !(((uintptr_t)fine | (uintptr_t)coarse) & 15)) {
        k_up_bwd8<<<grid_for(((long long)n * d * h * w) << cs), 256, 0, st>>>(fine, cf, f_off, coarse, cc, c_off, n, d, h, w, cs);
        return hipGetLastError();
    }
    k_up_bwd<<<grid_for((long long)n * d * h * w * c), 256, 0, st>>>(fine, cf, f_off, coarse, cc, c_off, n, d, h, w, c);
    return hipGetLastError();
}

hipError_t down_dgrad(const uint16_t *g, int cg, int g_off, const float *w, int cin, int cout, uint16_t *gx, int cx,
                      int x_off, int n, int d, int h, int wd, int accumulate, hipStream_t st)
{
    const long long nfine = (long long)n * d * h * wd;
    if (cin % 16 == 0 && cout % 16 == 0 && cin <= 128 && cg % 4 == 0 && g_off % 4 == 0 && nfine < 0x7fffffffLL &&
        ((uintptr_t)g & 7) == 0 && ((uintptr_t)w & 15) == 0) {
        const long long nvc = nfine / 8;
        const int nf = cin / 16 % 2 ? 1 : 2, ncb = cin / (16 * nf);
        const int mf = (nvc + 63) / 64 * ncb * 8 < 4096 ? 1 : 4;      // voxels per wave: 64, fewer on small grids
        const dim3 blocks((unsigned)(((nvc + 16 * mf - 1) / (16 * mf) * ncb + 3) / 4), 8);
        if (nf == 2 && mf == 4) k_down_dgrad_mfma<4, 2><<<blocks, 256, 0, st>>>(g, cg, g_off, w, cin, cout, gx, cx, x_off, n, d, h, wd, accumulate, ncb);
        else if (nf == 2) k_down_dgrad_mfma<1, 2><<<blocks, 256, 0, st>>>(g, cg, g_off, w, cin, cout, gx, cx, x_off, n, d, h, wd, accumulate, ncb);
        else if (mf == 4) k_down_dgrad_mfma<4, 1><<<blocks, 256, 0, st>>>(g, cg, g_off, w, cin, cout, gx, cx, x_off, n, d, h, wd, accumulate, ncb);
        else k_down_dgrad_mfma<1, 1><<<blocks, 256, 0, st>>>(g, cg, g_off, w, cin, cout, gx, cx, x_off, n, d, h, wd, accumulate, ncb);
        return hipGetLastError();
    }
    k_down_dgrad<<<grid_for(nfine * cin), 256, 0, st>>>(g, cg, g_off, w, cin, cout, gx, cx, x_off, n, d, h, wd, accumulate);
    return hipGetLastError();
}

hipError_t to_bf16(const float *x, int cs, long long nvox, int c, uint16_t *y, int cy, int y_off, int c_pad, hipStream_t st)
{
    const int ps = vec8(c_pad);
    if (ps >= 0 && cy % 8 == 0 && y_off % 8 == 0 && !((uintptr_t)y & 15)) {
        const int x4 = cs % 4 == 0 && !((uintptr_t)x & 15);
        k_to_bf16_8<<<grid_for(nvox << ps), 256, 0, st>>>(x, cs, nvox << ps, c, y, cy, y_off, ps, x4);
        return hipGetLastError();
    }
    k_to_bf16<<<grid_for(nvox * c_pad), 256, 0, st>>>(x, cs, nvox, c, y, cy, y_off, c_pad);
    return hipGetLastError();
}

hipError_t masked_mse(const float *pred, int cp, const float *target, const float *mask, long long nvox, int c,
                      uint16_t *g, int cg, float *loss_parts, int nparts, hipStream_t st)
{
    int *slot = (int *)(loss_parts + nparts);
    k_int_slot<<<1, 1, 0, st>>>(slot, 0);
    k_mask_count<<<grid_for(nvox), 256, 0, st>>>(mask, nvox, slot);
    k_masked_mse<<<nparts, 256, 0, st>>>(pred, cp, target, mask, nvox, c, loss_parts + nparts, g, cg, loss_parts);
    k_int_slot<<<1, 1, 0, st>>>(slot, 1);
    return hipGetLastError();
}

hipError_t bbox(const float *field, int cf, int n, int R, int *box, hipStream_t st)
{
    k_bbox<<<n, 256, 0, st>>>(field, cf, R, box);
    return hipGetLastError();
}

hipError_t crop_origin(const int *box, int n, int R, int D, int H, int W, int *origin, hipStream_t st)
{
    k_crop_origin<<<(n + 63) / 64, 64, 0, st>>>(box, n, R, D, H, W, origin);
    return hipGetLastError();
}

hipError_t crop(const float *src, int c, int n, int R, const int *origin, int D, int H, int W, float *dst, int uncrop,
                hipStream_t st)
{
    const long long per = uncrop ? (long long)R * R * R : (long long)D * H * W;
    k_crop<<<grid_for(per * n * c), 256, 0, st>>>(src, c, n, R, origin, D, H, W, dst, uncrop);
    return hipGetLastError();
}

hipError_t adam(const AdamJob *jobs, int count, float lr, float b1, float b2, float eps, int t, hipStream_t st)
{
    return launch_jobs(jobs, count, [](const AdamJob &j) { return (int)((j.n + 1023) / 1024); },
                       [&](const Jobs<AdamJob> &q, unsigned g) { k_adam<<<g, 256, 0, st>>>(q, lr, b1, b2, eps, t); });
}

}  // namespace nn
