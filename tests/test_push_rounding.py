"""Host check of the push's arithmetic: the Boris step and cosh / sinh of the
undulator field round as the divisions and square roots of their formulas do
(compiled for the host from the device header, bit for bit)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# what the device headers take from the HIP runtime, for a host compiler
STUB = r"""
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>
#define __device__
#define __host__
#define __global__
#define __shared__ static
#define __launch_bounds__(...)
#define amdgpu_waves_per_eu(...) unused
struct uint3 { unsigned x, y, z; };
static uint3 threadIdx, blockIdx, blockDim, gridDim;
struct int4 { int x, y, z, w; };
struct uint4 { unsigned x, y, z, w; };
inline int4 make_int4(int a, int b, int c, int d) { return {a, b, c, d}; }
typedef void *hipStream_t;
typedef int hipError_t;
template <class T> T min(T a, T b) { return b < a ? b : a; }
template <class T> T max(T a, T b) { return a < b ? b : a; }
template <class T> T __shfl_xor(T v, int) { return v; }
template <class T, class U> T atomicAdd(T *p, U v) { const T o = *p; *p += (T)v; return o; }
inline void __syncthreads() {}
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
inline int __builtin_amdgcn_update_dpp(int, int v, int, int, int, bool) { return v; }
inline int __builtin_amdgcn_readlane(int v, int) { return v; }
// the hardware's estimates: good to about 2^-26
inline double __builtin_amdgcn_rcp(double x) { return (1.0 / x) * (1.0 + 1.3e-8); }
inline double rsqrt(double x) { return 1.0 / std::sqrt(x); }
inline double cospi(double x) { return std::cos(3.14159265358979323846 * x); }
inline void sincospi(double x, double *s, double *c) { *s = std::sin(3.14159265358979323846 * x); *c = cospi(x); }
using std::isfinite;
"""

MAIN = r"""
#include "particle_dev.hpp"
#include <cstdio>
#include <random>
using namespace mithra;
int main()
{
    std::mt19937_64 g(7);
    std::uniform_real_distribution<double> U(-1.0, 1.0);
    long off = 0, offc = 0;
    for (int it = 0; it < 200000; ++it) {
        const double dtb = 1e-15 * (1.5 + U(g)), gam = 50.0 + 40.0 * U(g);
        RunDev R;
        memset((void *)&R, 0, sizeof R);
        R.ek = kQe * dtb / (2.0 * kMe * kC);
        R.ak = -kQe * dtb;
        double u[3], E[3], B[3], v[3];
        for (int a = 0; a < 3; ++a) {
            u[a] = v[a] = 2.0 * U(g);
            B[a] = gam * U(g);
            E[a] = gam * kC * U(g);
        }
        boris(R, u, E, B);
        double t1[3], t2[3];
        for (int a = 0; a < 3; ++a)
            t1[a] = v[a] - R.ek * E[a];
        const double al = -kQe * dtb / (2.0 * kMe * std::sqrt(1.0 + t1[0] * t1[0] + t1[1] * t1[1] + t1[2] * t1[2]));
        for (int a = 0; a < 3; ++a)
            t2[a] = t1[a] + al * (t1[(a + 1) % 3] * B[(a + 2) % 3] - t1[(a + 2) % 3] * B[(a + 1) % 3]);
        const double f = 2.0 * al / (1.0 + al * al * (B[0] * B[0] + B[1] * B[1] + B[2] * B[2]));
        const double s[3] = {f * B[0], f * B[1], f * B[2]};
        for (int a = 0; a < 3; ++a) {
            const double w = t1[a] + (t2[(a + 1) % 3] * s[(a + 2) % 3] - t2[(a + 2) % 3] * s[(a + 1) % 3]) - R.ek * E[a];
            off += w != u[a];
        }
        const double x = 3.0 * U(g);
        double ch, sh;
        cosh_sinh(x, ch, sh);
        const double em = std::expm1(std::fabs(x)), h = 0.5 * em / (1.0 + em);
        offc += sh != std::copysign(h * (2.0 + em), x) || ch != std::fma(h, em, 1.0);
    }
    std::printf("%ld %ld\n", off, offc);
}
"""


def test_boris_and_cosh_sinh_round_as_their_divisions(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(STUB)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "main")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-ffp-contract=off", f"-I{tmp_path}",
                    f"-I{ROOT}/paper_2009_13645_amd/csrc", f"-I{ROOT}/include", str(tmp_path / "main.cpp"),
                    "-o", exe], check=True)
    off, offc = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()
    assert int(off) == 0 and int(offc) == 0, (off, offc)
