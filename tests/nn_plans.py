"""The convolutions' tile planners (nn_plan.hpp) built for the host, for the tests."""
import ctypes as ct
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2302_04659_amd", "csrc")
CONV = ("TZ", "TX", "PW", "CW", "HZ", "HY", "HX", "tiles_x", "tiles_y", "tiles_z", "nco", "lds", "FR", "NF", "mTX", "mHX", "mHY")
WGRAD = ("TZ", "TX", "ns", "HX", "ncf", "nch", "nkh", "ncb", "ncg", "tiles_x", "tiles_y", "tiles_z", "tpg", "groups", "nvar",
         "g_off", "x_off", "lds", "mTX", "mHX", "mNP")
SOURCE = """
#include "%s/nn_plan.hpp"
static void sizes(int kind, int d, int h, int w, int &od, int &oh, int &ow)
{
    od = kind == 1 ? 2 * d : (kind == 2 ? d / 2 : d);
    oh = kind == 1 ? 2 * h : (kind == 2 ? h / 2 : h);
    ow = kind == 1 ? 2 * w : (kind == 2 ? w / 2 : w);
}
extern "C" int conv(int kind, int n, int d, int h, int w, int cin, int cout, unsigned *out)
{
    nn::ConvArgs a{};
    a.kind = kind; a.n = n; a.id = d; a.ih = h; a.iw = w; a.cx = a.cin = cin; a.cout = cout;
    sizes(kind, d, h, w, a.od, a.oh, a.ow);
    nn::ConvPlan p{};
    int FR = nn::FIRST_ROWS;
    const int NF = cout > 16 ? 2 : 1;
    if (!(cin == 8 ? nn::first_plan(a, p) : nn::conv_plan(a, NF, p, FR))) return 0;
    const unsigned v[] = {(unsigned)p.TZ, (unsigned)p.TX, (unsigned)p.PW, (unsigned)p.CW, (unsigned)p.HZ, (unsigned)p.HY,
                          (unsigned)p.HX, (unsigned)p.tiles_x, (unsigned)p.tiles_y, (unsigned)p.tiles_z, (unsigned)p.nco,
                          (unsigned)p.lds, (unsigned)FR, (unsigned)NF, p.mTX, p.mHX, p.mHY};
    for (unsigned i = 0; i < sizeof(v) / sizeof(v[0]); i++) out[i] = v[i];
    return 1;
}
extern "C" int wgrad(int kind, int n, int d, int h, int w, int cin, int cout, long long chunk, unsigned *out)
{
    nn::WgradArgs a{};
    a.kind = kind; a.n = n; a.id = d; a.ih = h; a.iw = w; a.cx = a.cin = cin; a.cg = a.cout = cout; a.chunk = chunk;
    sizes(kind, d, h, w, a.od, a.oh, a.ow);
    nn::WgradPlan p{};
    if (!nn::wgrad_plan(a, p)) return 0;
    const unsigned v[] = {(unsigned)p.TZ, (unsigned)p.TX, (unsigned)p.ns, (unsigned)p.HX, (unsigned)p.ncf, (unsigned)p.nch,
                          (unsigned)p.nkh, (unsigned)p.ncb, (unsigned)p.ncg, (unsigned)p.tiles_x, (unsigned)p.tiles_y,
                          (unsigned)p.tiles_z, (unsigned)p.tpg, (unsigned)p.groups, (unsigned)p.nvar, (unsigned)p.g_off,
                          (unsigned)p.x_off, (unsigned)p.lds, p.mTX, p.mHX, p.mNP};
    for (unsigned i = 0; i < sizeof(v) / sizeof(v[0]); i++) out[i] = v[i];
    return 1;
}
""" % CSRC


class Plans:
    def __init__(self, folder):
        src, lib = os.path.join(folder, "plans.cpp"), os.path.join(folder, "plans.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        # plain C++: a HIP object would register its (absent) device code with the GPU tests' process
        subprocess.run(["g++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-O1", "-std=c++17", "-fPIC", "-shared",
                        "-o", lib, src], check=True, capture_output=True)
        self.L = ct.CDLL(lib)

    def conv(self, kind, n, d, h, w, cin, cout):
        out = (ct.c_uint * len(CONV))()
        assert self.L.conv(kind, n, d, h, w, cin, cout, out) == 1
        return dict(zip(CONV, out))

    def wgrad(self, kind, n, d, h, w, cin, cout, chunk):
        out = (ct.c_uint * len(WGRAD))()
        assert self.L.wgrad(kind, n, d, h, w, cin, cout, ct.c_longlong(chunk), out) == 1
        return dict(zip(WGRAD, out))
