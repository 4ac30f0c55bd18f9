"""Samples with bits at or above n_qubits (latched as NQS_E_RANGE, but still
evaluated where pairs of samples are compared): the matrix elements read
nothing outside their tables.

The device functions are compiled here as plain C++ and run on the CPU over
tables that lie between guard values (NaN): a read outside a table makes the
element NaN.  In range, every element is the same number with and without the
stray bits, since these are not qubits.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_23809_amd", "csrc")
CLANG = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")

# What the device header takes from the HIP runtime, for one CPU thread.
SHIM = r"""
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#define __device__
#define __host__
#define __global__
#define __shared__ static
#define __forceinline__ inline
#define __noinline__
#define __launch_bounds__(...)
typedef int hipError_t;
typedef void *hipStream_t;
typedef void *hipEvent_t;
struct uint2 { unsigned x, y; };
struct uint4 { unsigned x, y, z, w; };
struct float2 { float x, y; };
struct double2 { double x, y; };
inline double2 make_double2(double a, double b) { return {a, b}; }
inline float2 make_float2(float a, float b) { return {a, b}; }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline int __popc(unsigned v) { return __builtin_popcount(v); }
inline float __uint_as_float(unsigned v) { float f; std::memcpy(&f, &v, 4); return f; }
inline unsigned __float_as_uint(float f) { unsigned v; std::memcpy(&v, &f, 4); return v; }
inline long long __double_as_longlong(double d) { long long v; std::memcpy(&v, &d, 8); return v; }
inline double __longlong_as_double(long long v) { double d; std::memcpy(&d, &v, 8); return d; }
template <class T> T __shfl(T v, int) { return v; }
template <class T> T atomicOr(T *p, T v) { T o = *p; *p = o | v; return o; }
template <class T> T atomicAdd(T *p, T v) { T o = *p; *p = o + v; return o; }
template <class T> T atomicCAS(T *p, T c, T v) { T o = *p; if (o == c) *p = v; return o; }
struct { unsigned x; } static threadIdx, blockIdx, blockDim;
using std::isfinite; using std::min; using std::max;
#define __builtin_amdgcn_readlane(v, l) (v)
#define __builtin_amdgcn_mbcnt_lo(a, b) (b)
#define __builtin_amdgcn_mbcnt_hi(a, b) (b)
"""

HEAD = r"""
#include <cstdio>
#include <vector>
#include "nqs_dev_common.hpp"
#include "nqs_table.hpp"
using namespace nqs;
// n values between two guards of NaN
struct Guarded {
    std::vector<double> all;
    size_t pad;
    Guarded(const std::vector<double> &v, size_t p) : all(v.size() + 2 * p, __builtin_nan("")), pad(p) {
        std::copy(v.begin(), v.end(), all.begin() + p);
    }
    const double *data() const { return all.data() + pad; }
};
static uint64_t state = 88172645463325252ull;
static uint64_t rnd() { state ^= state << 13; state ^= state >> 7; return state ^= state << 17; }
static double uniform() { return static_cast<double>(rnd() >> 11) / 9007199254740992.0 - 0.5; }
static int bad = 0;
static void expect(bool ok, const char *what, int nq) {
    if (!ok && ++bad < 5) std::printf("%s, %d qubits\n", what, nq);
}
// a sample of the register and bits outside it (none for stray = 0)
template <int W>
static Key<W> sample(int nq, uint64_t stray) {
    Key<W> k;
    uint64_t w[2];
    for (int q = 0; q < 2; ++q) {
        const int b = nq - 64 * q;
        const uint64_t in = b >= 64 ? ~0ull : b > 0 ? (1ull << b) - 1 : 0ull;
        w[q] = (rnd() & in) | (stray & ~in);
    }
    for (int q = 0; q < W; ++q) k.w[q] = w[q];
    return k;
}
template <int W>
static Key<W> outside(Key<W> k, int nq, uint64_t stray) {
    for (int q = 0; q < W; ++q) {
        const int b = nq - 64 * q;
        const uint64_t in = b >= 64 ? ~0ull : b > 0 ? (1ull << b) - 1 : 0ull;
        k.w[q] = (k.w[q] & in) | (stray & ~in);
    }
    return k;
}
"""

INTEGRALS = r"""
template <int W>
static void run(int K) {
    const int nq = 2 * K;
    std::vector<double> h(size_t(K) * K), e;
    for (double &v : h) v = uniform();
    const size_t np = size_t(K) * (K + 1) / 2;
    e.resize(np * (np + 1) / 2);
    for (double &v : e) v = uniform();
    // (orbitals to 63: the largest index such a pair could form)
    const Guarded gh(h, 64 * 64), ge(e, 64 * 65 / 2 * (64 * 65 / 2 + 1) / 2);
    DevTable tab{};
    tab.n_qubits = nq;
    tab.sc = 1;
    tab.sc_k = K;
    tab.sc_h1 = gh.data();
    tab.sc_eri = ge.data();
    for (int k = 0; k < 4000; ++k) {
        Key<W> x = sample<W>(nq, 0), y = x;
        // one to four flips: a single, a double or neither
        for (int f = 0; f < 1 + k % 4; ++f) flip_bit<W>(y, static_cast<int>(rnd() % nq));
        const double v = sc_element<W>(tab, x, y);
        expect(v == v, "element of valid samples", nq);
        const uint64_t s = rnd();
        const double a = sc_element<W>(tab, outside<W>(x, nq, s), outside<W>(y, nq, s));
        expect(a == v, "element, both with the same stray bits", nq);
        const double b = sc_element<W>(tab, outside<W>(x, nq, rnd()), outside<W>(y, nq, rnd()));
        expect(b == v, "element, with different stray bits", nq);
        // pairs that differ in stray bits alone
        const Key<W> z = outside<W>(x, nq, s ^ (3ull << 61) ^ (k & 1 ? 5ull << 56 : 0ull));
        expect(sc_element<W>(tab, outside<W>(x, nq, s), z) == 0.0, "element across stray bits", nq);
        const double d = sc_diagonal<W>(tab, x);
        expect(d == d && sc_diagonal<W>(tab, outside<W>(x, nq, s)) == d, "diagonal", nq);
    }
}
int main() {
    run<1>(2); run<1>(6); run<1>(20); run<1>(31); run<2>(32); run<2>(33); run<2>(50); run<2>(63);
    if (bad) std::printf("%d wrong\n", bad);
    return bad != 0;
}
"""


def check(tmp_path, body):
    if not os.path.exists(CLANG):
        pytest.skip("no ROCm clang++")
    os.makedirs(tmp_path / "hip")
    (tmp_path / "hip" / "hip_runtime.h").write_text(SHIM)
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(HEAD + body)
    subprocess.check_call([CLANG, "-std=c++17", "-O1", "-w", f"-I{tmp_path}", f"-I{CSRC}", str(src),
                           os.path.join(CSRC, "nqs_table.cpp"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr


def test_integral_elements_stay_inside_their_tables(tmp_path):
    check(tmp_path, INTEGRALS)


ROWS = r"""
// one group of one or two flips whose strings differ from a base in one qubit
// (an occupation row), the last piece of its table, and a tabulated one
template <int W>
static void run(int nq, int flips) {
    std::vector<uint64_t> x, z;
    std::vector<double> c;
    const auto term = [&](uint64_t z0, uint64_t z1) {
        uint64_t X[2] = {0, 0};
        for (int f = 0; f < flips; ++f) X[(3 * f) >> 6] |= 1ull << (3 * f);
        x.insert(x.end(), X, X + 2);
        z.push_back(z0);
        z.push_back(z1);
        c.push_back(uniform());
    };
    for (int q = 0; q < nq; ++q)
        if (q % 3 || q >= 3 * flips) term(q < 64 ? 1ull << q : 0, q < 64 ? 0 : 1ull << (q - 64));
    // (the string of the base balances them: the row form is kept)
    double sum = 0.0;
    for (const double v : c) sum += v;
    term(0, 0);
    c.back() = -sum;
    HostTable T;
    std::string err;
    if (build_table(nq, static_cast<int64_t>(c.size()), x.data(), z.data(), c.data(), nullptr, &T, &err)) {
        std::printf("%s\n", err.c_str());
        ++bad;
        return;
    }
    GroupRecords R;
    build_group_records(T, &R);
    expect(R.rows.size() == 2 * size_t(nq + 2), "one occupation row", nq);
    const Guarded rows(R.rows, 256);
    std::vector<uint32_t> goff(T.goff.begin(), T.goff.end());
    DevTable tab{};
    tab.n_qubits = nq;
    tab.gx = R.rec.data();
    tab.gx_stride = kGroupWords;
    tab.goff = goff.data();
    tab.tz = R.z.data();
    tab.tc = T.tc.data();
    tab.tcode = R.codes.data();
    tab.occ = rows.data();
    for (int k = 0; k < 2000; ++k) {
        unsigned long long terms = 0;
        const Key<W> s = sample<W>(nq, 0);
        const double v = group_sum<W, false>(tab, 0, s, nullptr, &terms);
        expect(v == v, "sum of a valid sample", nq);
        expect(group_sum<W, false>(tab, 0, outside<W>(s, nq, rnd()), nullptr, &terms) == v,
               "sum with stray bits", nq);
        expect(group_sum<W, false>(tab, 0, outside<W>(s, nq, ~0ull), nullptr, &terms) == v,
               "sum with all stray bits", nq);
    }
}
int main() {
    for (int f = 1; f <= 2; ++f) {
        run<1>(12, f); run<1>(24, f); run<1>(62, f); run<1>(63, f);
        run<2>(64, f); run<2>(66, f); run<2>(100, f); run<2>(127, f);
    }
    if (bad) std::printf("%d wrong\n", bad);
    return bad != 0;
}
"""


def test_occupation_rows_stay_inside_their_tables(tmp_path):
    check(tmp_path, ROWS)
