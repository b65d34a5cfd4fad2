// Tiles and wave splits of the surrogate's convolutions (internal, host): what a
// launch of k_conv_pos, k_conv_first or k_wgrad is cut into.
#pragma once
#include <algorithm>
#include <cmath>

#include "nn_kernels.hpp"

namespace nn {

struct ConvPlan {
    int TZ, TX, PW, CW;            // tile positions, waves along positions and output channels
    int HZ, HY, HX;                // halo extents
    int tiles_x, tiles_y, tiles_z, ntiles, nco;
    unsigned mTX, mHX, mHY;        // reciprocals ceil(2^32 / d)
    int x16, wide, lds;            // 16-byte copies possible; boxes of over 2^32 voxels
};

constexpr int FIRST_ROWS = 4;   // output rows (y) of a first-layer tile
constexpr int WTY = 4;          // output rows (y) of a weight-gradient tile

struct WgradPlan {
    int TZ, TX, ns, HX;            // tile positions (z, x), K steps of 32 positions, X row length (even)
    int ncf, nch, nkh, ncb, ncg;   // wave split; blocks of input channels, groups of output channels
    int tiles_x, tiles_y, tiles_z, ntiles, tpg, groups, nvar;
    unsigned mTX, mHX, mNP;        // reciprocals ceil(2^32 / d) of TX, HX and 32 ns
    int g_off, x_off, lds;         // byte offsets of the G and X tiles, LDS bytes
    int x16, g16, wide;            // 16-byte copies possible; boxes of over 2^32 voxels
};

// Sizes of a tile along an axis of n worth looking at: n cut into 1, 2, 3, ... even parts.
inline int next_cut(int n, int t)   // the next smaller one, 0 at the end
{
    if (t <= 1) return 0;
    const int k = (n + t - 1) / t;
    for (int m = k + 1;; m++) {
        const int u = (n + m - 1) / m;
        if (u < t) return u;
    }
}

inline unsigned recip(int d) { return (unsigned)((0x100000000ull + d - 1) / d); }

// Tile, rows per wave and wave split of a convolution with the least estimated
// time, in clocks: a compute unit's share of the workgroups times the sum of
// their MFMAs (20 clocks each on the four SIMDs, 16 at the peak, times the
// busiest SIMD's share of the waves), halo bytes (10 a clock) and output bytes
// (20 a clock), 15 % more with fewer than three workgroups per CU to overlap
// these phases; or, where few workgroups are in flight, the rounds of one
// workgroup's own chain (900 clocks of latency per (z, x) tap, 4,500 per
// chunk).  Fitted to a sweep of 1,548 tiles over ten layers (32 to 128
// channels, 8 and 64 boxes of 40 x 24 x 40 and their two coarser levels): the
// tiles it picks are within 9 % of the fastest of each.
inline bool conv_plan(const ConvArgs &a, int NF, ConvPlan &p, int &FR)
{
    const bool up = a.kind == KIND_UP;
    const int kc = a.cin / 32, groups = (a.cout + 16 * NF - 1) / (16 * NF);
    double best = -1.0;
    for (int fr : {8, 6, 4}) {
        const int HY = up ? fr / 2 + 2 : fr + 2;
        for (int TX = a.ow; TX > 0; TX = next_cut(a.ow, TX))
            for (int TZ = a.od; TZ > 0; TZ = next_cut(a.od, TZ)) {
                if (TX > 128 || TZ * TX > 128) continue;
                const int PW = (TZ * TX + 15) / 16;
                const int HX = up ? TX / 2 + 2 : TX + 2, HZ = up ? TZ / 2 + 2 : TZ + 2;
                const int hb = 64 * HZ * HY * HX;
                const double tiles = (double)a.n * ((a.ow + TX - 1) / TX) * ((a.oh + fr - 1) / fr) * ((a.od + TZ - 1) / TZ);
                for (int CW = groups; CW >= 1; CW /= 2) {
                    const int most = NF == 2 && fr == 8 ? 8 : 16;   // waves, as the launch bounds
                    if (PW * CW > most) continue;
                    const int lds = hb;
                    if (lds > 80 * 1024) continue;                    // two workgroups per CU; a launch may ask for 160 KB
                    const int occ = std::min(160 * 1024 / lds, std::max(1, (most == 8 ? 12 : 16) / (PW * CW)));
                    const double wgs = tiles * (groups / CW);
                    const int W = PW * CW;
                    const double mf = 27.0 * fr * NF * ((occ * W + 3) / 4) / occ, out = 16.0 * W * fr * 32 * NF;
                    const double all = (kc * (20 * mf + hb / 10.0) + out / 20) * (occ < 3 ? 1.15 : 1.0);
                    const double own = kc * (9 * (900.0 + 48 * fr * NF * ((W + 3) / 4)) + hb / 10.0 + 4500.0) + 2000.0;
                    const double cost = std::max(std::ceil(wgs / 256) * all, std::ceil(wgs / (256.0 * occ)) * own);
                    if (best >= 0.0 && cost >= best) continue;
                    best = cost;
                    FR = fr;
                    p.TZ = TZ; p.TX = TX; p.PW = PW; p.CW = CW;
                    p.HZ = HZ; p.HY = HY; p.HX = HX;
                    p.lds = lds;
                    p.nco = groups / CW;
                }
            }
    }
    if (best < 0.0) return false;
    p.tiles_x = (a.ow + p.TX - 1) / p.TX;
    p.tiles_y = (a.oh + FR - 1) / FR;
    p.tiles_z = (a.od + p.TZ - 1) / p.TZ;
    const long long nt = (long long)a.n * p.tiles_x * p.tiles_y * p.tiles_z;
    if ((nt + 7) * p.nco > 0x7fffffff) return false;
    p.ntiles = (int)nt;
    p.mTX = recip(p.TX);
    p.mHX = recip(p.HX);
    p.mHY = recip(p.HY);
    p.wide = VoxelIndex::needs_wide(a.id, a.ih, a.iw);
    p.x16 = a.cx % 8 == 0 && a.x_off % 8 == 0 && ((uintptr_t)a.x & 15) == 0;
    return true;
}

// Tile of the first layer: the least padded positions, then the smallest halo.
inline bool first_plan(const ConvArgs &a, ConvPlan &p)
{
    double best = -1.0;
    for (int TX = a.ow; TX > 0; TX = next_cut(a.ow, TX))
        for (int TZ = a.od; TZ > 0; TZ = next_cut(a.od, TZ)) {
            if (TX > 64 || TZ * TX > 64) continue;
            const double tiles = (double)((a.ow + TX - 1) / TX) * ((a.od + TZ - 1) / TZ);
            const double cost = tiles * (64 * 32 + 2.0 * (TZ + 2) * (TX + 2));
            if (best >= 0.0 && cost >= best) continue;
            best = cost;
            p.TX = TX; p.TZ = TZ;
        }
    p.HX = p.TX + 2; p.HZ = p.TZ + 2; p.HY = FIRST_ROWS + 2;
    p.tiles_x = (a.ow + p.TX - 1) / p.TX;
    p.tiles_y = (a.oh + FIRST_ROWS - 1) / FIRST_ROWS;
    p.tiles_z = (a.od + p.TZ - 1) / p.TZ;
    const long long nt = (long long)a.n * p.tiles_x * p.tiles_y * p.tiles_z;
    if (nt > 0x7ffffff0) return false;
    p.ntiles = (int)nt;
    p.mTX = recip(p.TX);
    p.mHX = recip(p.HX);
    p.lds = 16 * p.HZ * p.HY * p.HX;
    p.wide = VoxelIndex::needs_wide(a.id, a.ih, a.iw);
    return true;
}

// Tile and wave split of a weight gradient: the tile shape (z, x positions)
// with the least estimated time, MFMA steps (16 clocks per MFMA, four waves on
// four SIMDs, padding positions included) plus the staged bytes at the 32
// bytes per clock and CU a workgroup's copies reach, within 60 KB of LDS (two
// workgroups per CU).  Larger tiles waste positions on small grids, smaller
// ones stage more halo.
inline bool wgrad_plan(const WgradArgs &a, WgradPlan &p)
{
    const int NT = a.kind == KIND_C3 || a.kind == KIND_UP ? 3 : (a.kind == KIND_DOWN ? 2 : 1);
    const int S = a.kind == KIND_DOWN ? 2 : 1, RY = S * (WTY - 1) + NT;
    const int nf = (a.cout + 15) / 16, NF = nf >= 2 ? 2 : 1;
    p.ncf = a.cin >= 32 ? 2 : 1;
    p.nch = nf >= 4 ? 2 : 1;
    p.nkh = 4 / (p.ncf * p.nch);
    p.ncb = (a.cin + 16 * p.ncf - 1) / (16 * p.ncf);
    p.ncg = (nf + NF * p.nch - 1) / (NF * p.nch);
    p.nvar = NT * p.ncb * p.ncg;
    const int xrow = 32 * p.ncf, grow = 32 * NF * p.nch;
    const int red = p.nkh > 1 ? p.ncf * p.nch * NT * NT * NF * 1024 : 0;
    double best = -1.0;
    for (int TX = a.ow; TX > 0; TX = next_cut(a.ow, TX))
        for (int TZ = a.od; TZ > 0; TZ = next_cut(a.od, TZ)) {
            if (TX > 96 || TZ * TX > 96) continue;
            const int ns = (TZ * TX + 31) / 32, HX = (S * (TX - 1) + NT + 1) & ~1;
            const int tab = 128 * ns, gb = WTY * 32 * ns * grow, xb = TZ * RY * HX * xrow;
            if (tab + gb + xb > 60 * 1024) continue;
            const double steps = (double)((ns + p.nkh - 1) / p.nkh) * NT * NT * WTY * NF * 16;
            const double cost = (double)((a.ow + TX - 1) / TX) * ((a.od + TZ - 1) / TZ) * (steps + (gb + xb) / 32.0 + 200.0);
            if (best >= 0.0 && cost >= best) continue;
            best = cost;
            p.TX = TX; p.TZ = TZ; p.ns = ns; p.HX = HX;
            p.g_off = tab;
            p.x_off = tab + gb;
            p.lds = tab + gb + xb > red ? tab + gb + xb : red;
        }
    if (best < 0.0) return false;
    p.mTX = recip(p.TX);
    p.mHX = recip(p.HX);
    p.mNP = recip(32 * p.ns);
    p.tiles_x = (a.ow + p.TX - 1) / p.TX;
    p.tiles_y = (a.oh + WTY - 1) / WTY;
    p.tiles_z = (a.od + p.TZ - 1) / p.TZ;
    const long long nvox = (long long)a.n * a.od * a.oh * a.ow;
    const long long ntiles = (long long)a.n * p.tiles_x * p.tiles_y * p.tiles_z;
    const long long groups_max = (nvox + a.chunk - 1) / a.chunk;          // the partial buffer holds this many
    // about three workgroups per CU over all variants; every group adds a partial to write and to sum
    const long long want = std::min(groups_max, std::max(1LL, 768LL / p.nvar));
    const long long tpg = (ntiles + want - 1) / want, groups = (ntiles + tpg - 1) / tpg;
    if (ntiles > 0x7fffffff || (groups + 8) * p.nvar > 0x7fffffff) return false;
    p.ntiles = (int)ntiles;
    p.tpg = (int)tpg;
    p.groups = (int)groups;
    p.wide = VoxelIndex::needs_wide(a.id, a.ih, a.iw) || VoxelIndex::needs_wide(a.od, a.oh, a.ow);
    p.x16 = a.cx % 8 == 0 && a.x_off % 8 == 0 && ((uintptr_t)a.x & 15) == 0;
    p.g16 = a.cg % 8 == 0 && a.g_off % 8 == 0 && a.cout % 8 == 0 && ((uintptr_t)a.g & 15) == 0;
    return true;
}

}  // namespace nn
