// Device helpers shared by the kernel translation units: sample keys,
// the linear hash and Bloom bits, the bucketed sample hash, the group
// index, group term sums (FP64 and FP32 with compensation), the
// Slater-Condon element and the FP32 amplitude ratio.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/nqs.h"
#include "nqs_device.hpp"

namespace nqs {

// ------------------------------------------------------------------ helpers

template <int W>
struct Key {
    uint64_t w[W];
};

template <int W>
__device__ __forceinline__ Key<W> load_key(const uint64_t *__restrict__ p, int64_t i) {
    Key<W> k;
#pragma unroll
    for (int q = 0; q < W; ++q) k.w[q] = p[2 * i + q];
    return k;
}

// The bits of k below n_qubits.  A sample with others is latched as an error
// but still compared with the rest of its batch, so whatever turns set bits
// into indices of a table takes these alone.
template <int W>
__device__ __forceinline__ Key<W> in_register(const DevTable &tab, Key<W> k) {
    if constexpr (W == 1) {
        k.w[0] &= (1ull << tab.n_qubits) - 1ull;
    } else {
        k.w[W - 1] &= (1ull << (tab.n_qubits - 64)) - 1ull;
    }
    return k;
}

template <int W>
__device__ __forceinline__ uint32_t linear_hash(const Key<W> &k, const uint32_t *__restrict__ hr) {
    uint32_t h = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        uint64_t v = k.w[q];
        while (v) {
            h ^= hr[64 * q + __builtin_ctzll(v)];
            v &= v - 1;
        }
    }
    return h;
}

// Bits of x selected by (m0, m1), packed to the low end in mask order.
template <int W>
__device__ __forceinline__ uint64_t compress(const Key<W> &x, uint64_t m0, uint64_t m1) {
    uint64_t r = 0;
    int k = 0;
    while (m0) {
        const int b = __builtin_ctzll(m0);
        r |= ((x.w[0] >> b) & 1ull) << k++;
        m0 &= m0 - 1;
    }
    if constexpr (W == 2) {
        while (m1) {
            const int b = __builtin_ctzll(m1);
            r |= ((x.w[1] >> b) & 1ull) << k++;
            m1 &= m1 - 1;
        }
    }
    return r;
}

__device__ __forceinline__ uint32_t slot_of(uint32_t h, uint32_t shift) {
    return (h * kGoldenMul) >> shift;
}

// One bucket of the sample hash: 64 bytes of keys (8 one-word or 4
// two-word), four independent 16-byte loads.
struct Bucket {
    uint4 q0, q1, q2, q3;
};

template <int W>
__device__ __forceinline__ Bucket bucket_load(const uint64_t *__restrict__ skey, uint32_t start) {
    const uint4 *p = reinterpret_cast<const uint4 *>(skey + static_cast<size_t>(start) * W);
    return Bucket{p[0], p[1], p[2], p[3]};
}

// Slot of the bucket holding k (or -1), and whether the bucket has a free
// slot.  Occupied slots form a prefix of a bucket (a key takes the first
// free slot from its start on, and nothing is removed), so the bucket is
// open iff its last slot is free; a key is stored once, so any slot that
// matches is the one.  The common case (no match) costs one XOR-OR per key
// word and a minimum.
template <int W>
__device__ __forceinline__ uint32_t slot_diff(const Bucket &b, int s, const Key<W> &k) {
    // zero iff slot s holds k (s a compile-time constant after unrolling)
    const uint32_t k0l = static_cast<uint32_t>(k.w[0]), k0h = static_cast<uint32_t>(k.w[0] >> 32);
    if constexpr (W == 1) {
        const uint4 &v = (s >> 1) == 0 ? b.q0 : (s >> 1) == 1 ? b.q1 : (s >> 1) == 2 ? b.q2 : b.q3;
        return (s & 1) ? ((v.z ^ k0l) | (v.w ^ k0h)) : ((v.x ^ k0l) | (v.y ^ k0h));
    } else {
        const uint32_t k1l = static_cast<uint32_t>(k.w[1]), k1h = static_cast<uint32_t>(k.w[1] >> 32);
        const uint4 &v = s == 0 ? b.q0 : s == 1 ? b.q1 : s == 2 ? b.q2 : b.q3;
        return (v.x ^ k0l) | (v.y ^ k0h) | (v.z ^ k1l) | (v.w ^ k1h);
    }
}

template <int W>
__device__ __forceinline__ int bucket_scan(const Bucket &b, const Key<W> &k, bool &empty) {
    constexpr int BK = 1 << bucket_log2(W);
    // the last slot's key (its last word) is the bucket's last word
    empty = (b.q3.z & b.q3.w) == 0xFFFFFFFFu;
    uint32_t m = slot_diff<W>(b, 0, k);
#pragma unroll
    for (int s = 1; s < BK; ++s) m = min(m, slot_diff<W>(b, s, k));
    if (m != 0u) return -1;
    // a match (rare): which slot
    int found = 0;
#pragma unroll
    for (int s = BK - 1; s > 0; --s)
        if (slot_diff<W>(b, s, k) == 0u) found = s;
    return found;
}

// Index of key k in the sample hash, or -1, with the bucket at start already
// loaded (b); the index array is read only for the slot that holds the key.
template <int W>
__device__ __forceinline__ int32_t hash_find_from(const uint64_t *__restrict__ skey,
                                                  const int32_t *__restrict__ sidx, uint32_t mask,
                                                  uint32_t start, const Key<W> &k, Bucket b) {
    constexpr int BK = 1 << bucket_log2(W);
    for (uint32_t probe = 0; probe <= mask; probe += BK) {
        bool empty;
        const int found = bucket_scan<W>(b, k, empty);
        if (found >= 0) return sidx[(start + static_cast<uint32_t>(found)) & mask];
        if (empty) return -1;
        start = (start + BK) & mask;
        b = bucket_load<W>(skey, start);
    }
    return -1;
}

// Index of key in the sample hash, or -1 (one memory round trip per bucket).
template <int W>
__device__ __forceinline__ int32_t hash_find(const uint64_t *__restrict__ skey,
                                             const int32_t *__restrict__ sidx, uint32_t mask,
                                             uint32_t start, const Key<W> &k) {
    return hash_find_from<W>(skey, sidx, mask, start, k, bucket_load<W>(skey, start));
}

__device__ __forceinline__ void latch(int *err, int code) { atomicCAS(err, 0, code); }

__device__ __forceinline__ double readlane_f64(double v, int lane) {
    const uint64_t u = static_cast<uint64_t>(__double_as_longlong(v));
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(u), lane);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(u >> 32), lane);
    return __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi) << 32) | lo));
}

__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, int lane) {
    const uint32_t lo = __shfl(static_cast<uint32_t>(v), lane);
    const uint32_t hi = __shfl(static_cast<uint32_t>(v >> 32), lane);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ double shfl_f64(double v, int lane) {
    return __longlong_as_double(static_cast<long long>(
        shfl_u64(static_cast<uint64_t>(__double_as_longlong(v)), lane)));
}

typedef int v8i __attribute__((ext_vector_type(8)));

// 32 bits as FP4 -1 (0: 0x2 is +1, the sign bit set is -1), bits 4 k + c in
// nibble k of word c: the operand of a product over qubits in any order.
__device__ __forceinline__ v8i fp4_signs(uint32_t v) {
    v8i r = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < 4; ++c)
        r[c] = static_cast<int>(((v << (3 - c)) & 0x88888888u) | 0x22222222u);
    return r;
}

// Number of set bits of mask below this lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// Blocked Bloom filter of the sample hashes: a key with hash h sets two bits
// of one 32-bit word, word (h >> 2) & (words - 1) and bits (h >> 17) & 31 and
// (h >> 24) & 31 (disjoint ranges of h for filters of up to 2^15 words).  The
// byte offset of the word is h & ((words - 1) << 2), which folds into the
// XOR forming h; the shift by (h >> 24) reads byte 3 of h in place (a
// sub-dword operand), so a probe costs one shift less.
__device__ __forceinline__ uint32_t filter_word(uint32_t h, uint32_t wmask) {
    return (h >> 2) & wmask;
}
__device__ __forceinline__ uint32_t filter_bits(uint32_t h) {
    return (1u << ((h >> 17) & 31)) | (1u << ((h >> 24) & 31));
}
__device__ __forceinline__ uint32_t filter_test(uint32_t fw, uint32_t h) {
    return (fw >> ((h >> 17) & 31)) & (fw >> ((h >> 24) & 31)) & 1u;
}

// Word q of group g's flip mask.
template <int W>
__device__ __forceinline__ uint64_t group_x(const DevTable &tab, int64_t g, int q) {
    const uint64_t v = tab.gx[static_cast<size_t>(tab.gx_stride) * g + q];
    return q == W - 1 ? v & ~kGroupGeneral : v;
}

// The bits of x at the flips X (at most four, lowest first), and their number.
template <int W>
__device__ __forceinline__ uint32_t flip_pattern(const Key<W> &X, const Key<W> &x, int &m) {
    uint64_t lo = X.w[0], hi = W == 2 ? X.w[W - 1] : 0ull;
    uint32_t pat = 0;
    m = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if constexpr (W == 1) {
            const uint64_t b = lo & (0ull - lo);
            lo ^= b;
            m += b != 0ull;
            pat |= (x.w[0] & b) ? 1u << k : 0u;
        } else {
            const bool low = lo != 0ull;
            const uint64_t v = low ? lo : hi, b = v & (0ull - v);
            const uint64_t c = v ^ b;
            lo = low ? c : lo;
            hi = low ? hi : c;
            m += b != 0ull;
            pat |= ((low ? x.w[0] : x.w[W - 1]) & b) ? 1u << k : 0u;
        }
    }
    return pat;
}

// Sum of one group's terms for bra x, sum_t c~_t (-1)^{popc(Z_t & x)}: from
// the group's record where it is tabulated, from its occupation row where it
// has one, else term by term.  cnt: the group's terms if known (0 or 255:
// not).  One record of 64 bytes a hit instead of two arrays of 4 to 6 terms,
// or of 78 (198 at 100 qubits) for a single excitation.
template <int W, bool DUMP>
__device__ __forceinline__ double group_sum(const DevTable &tab, int64_t g, const Key<W> &x,
                                            uint32_t *__restrict__ sign_row,
                                            unsigned long long *terms, uint32_t cnt = 0) {
    if (cnt == 0u || cnt == 255u) cnt = tab.goff[g + 1] - tab.goff[g];
    *terms += cnt;
    const uint64_t *rec = tab.gx + static_cast<size_t>(kGroupWords) * g;
    const uint64_t *value = rec + 2 * W;
    Key<W> X;
    int par = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        X.w[q] = rec[q];
        par += __popcll(rec[W + q] & x.w[q]);
    }
    const bool general = (X.w[W - 1] & kGroupGeneral) != 0ull;
    X.w[W - 1] &= ~kGroupGeneral;
    double s = 0.0;
    if (!general) {
        int m;
        const uint32_t pat = flip_pattern<W>(X, x, m);
        // relative to the first flip
        const uint32_t rel = ((pat & 1u) ? ~pat : pat) & ((1u << m) - 1u);
        if constexpr (DUMP) {
            if (sign_row) {
                const uint32_t t0 = tab.goff[g];
                for (uint32_t t = t0; t < t0 + cnt; ++t)
                    if ((par + __popc(tab.tcode[t] & pat)) & 1)
                        atomicOr(&sign_row[t >> 5], 1u << (t & 31));
            }
        }
        if (m == 4 && (__popc(rel) & 1)) {
            // odd parity (samples of several sectors): the terms
            const uint32_t t0 = tab.goff[g];
            for (uint32_t t = t0; t < t0 + cnt; ++t)
                s += (__popc(tab.tcode[t] & rel) & 1) ? -tab.tc[t] : tab.tc[t];
        } else {
            s = reinterpret_cast<const double *>(value)[(rel >> 1) & 3u];
        }
        return (par & 1) ? -s : s;
    }
    if (!DUMP && value[2] != 0ull) {
        // occupied qubits four at a time (the last entry of a row is 0)
        const int nq = tab.n_qubits;
        const Key<W> occ = in_register<W>(tab, x);
        uint64_t lo = occ.w[0], hi = W == 2 ? occ.w[W - 1] : 0ull;
        int in = 0;  // flips of X that are occupied
#pragma unroll
        for (int q = 0; q < W; ++q) in += __popcll(X.w[q] & x.w[q]);
        const double *row = tab.occ + (2 * (value[2] - 1ull) + (in & 1)) * (nq + 2);
        s = row[0];
        while (lo | hi) {
            double v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                int at = nq + 1;
                if constexpr (W == 1) {
                    if (lo) at = 1 + __builtin_ctzll(lo);
                    lo &= lo - 1;
                } else {
                    const bool low = lo != 0ull;
                    const uint64_t b = low ? lo : hi;
                    if (b) at = (low ? 1 : 65) + __builtin_ctzll(b);
                    const uint64_t c = b & (b - 1);
                    lo = low ? c : lo;
                    hi = low ? hi : c;
                }
                v[k] = row[at];
            }
            s += v[0];
            s += v[1];
            s += v[2];
            s += v[3];
        }
        return (par & 1) ? -s : s;
    }
    const uint32_t t0 = tab.goff[g];
    const uint64_t *z = tab.tz + 2 * value[3];
    for (uint32_t k = 0; k < cnt; ++k) {
        int odd = 0;
#pragma unroll
        for (int q = 0; q < W; ++q) odd += __popcll(z[2 * static_cast<size_t>(k) + q] & x.w[q]);
        const double c = tab.tc[t0 + k];
        s += (odd & 1) ? -c : c;
        if constexpr (DUMP) {
            const uint32_t t = t0 + k;
            if (sign_row && (odd & 1)) atomicOr(&sign_row[t >> 5], 1u << (t & 31));
        }
    }
    return s;
}

// ---- integral form (Slater-Condon rules, the evaluator of Sec. III-B)
//
// <bra|H|ket> from h_pq and the chemists' (pq|rs) for determinants that
// differ by at most two spin orbitals; ONV ordering, so a ladder operator on
// spin orbital j carries (-1)^(occupied orbitals below j).

template <int W>
__device__ __forceinline__ int parity_below(const Key<W> &s, int j) {
    int c;
    if (j < 64) {
        c = __popcll(s.w[0] & ((1ull << j) - 1ull));
    } else {
        c = __popcll(s.w[0]);
        if constexpr (W == 2) c += __popcll(s.w[1] & ((1ull << (j - 64)) - 1ull));
    }
    return c & 1;
}

template <int W>
__device__ __forceinline__ void flip_bit(Key<W> &s, int j) {
    if (W == 1 || j < 64)
        s.w[0] ^= 1ull << (j & 63);
    else
        s.w[W - 1] ^= 1ull << (j & 63);
}

template <int W>
__device__ __forceinline__ int lowest(const Key<W> &s) {
    if (s.w[0]) return __builtin_ctzll(s.w[0]);
    if constexpr (W == 2) return 64 + __builtin_ctzll(s.w[1]);
    return 127;
}

__device__ __forceinline__ double eri_at(const DevTable &tab, int p, int q, int r, int s) {
    const int64_t pq = p > q ? int64_t(p) * (p + 1) / 2 + q : int64_t(q) * (q + 1) / 2 + p;
    const int64_t rs = r > s ? int64_t(r) * (r + 1) / 2 + s : int64_t(s) * (s + 1) / 2 + r;
    return tab.sc_eri[pq > rs ? pq * (pq + 1) / 2 + rs : rs * (rs + 1) / 2 + pq];
}

template <int W>
__device__ __forceinline__ double sc_element(const DevTable &tab, const Key<W> &b_any,
                                             const Key<W> &k_any) {
    const Key<W> bra = in_register<W>(tab, b_any), ket = in_register<W>(tab, k_any);
    Key<W> A, I;
    int na = 0, ni = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        A.w[q] = bra.w[q] & ~ket.w[q];  // created
        I.w[q] = ket.w[q] & ~bra.w[q];  // annihilated
        na += __popcll(A.w[q]);
        ni += __popcll(I.w[q]);
    }
    if (na != ni) return 0.0;
    const int K = tab.sc_k;
    if (na == 1) {
        const int i = lowest<W>(I), a = lowest<W>(A);
        if ((i & 1) != (a & 1)) return 0.0;
        Key<W> st = ket;
        int sg = parity_below<W>(st, i);
        flip_bit<W>(st, i);
        sg ^= parity_below<W>(st, a);
        const int as = a >> 1, is = i >> 1;
        double v = tab.sc_h1[as * K + is];
        // spectators: occupied in ket, except i
#pragma unroll
        for (int q = 0; q < W; ++q) {
            uint64_t m = ket.w[q] & ~I.w[q];
            while (m) {
                const int j = 64 * q + __builtin_ctzll(m);
                m &= m - 1;
                const int js = j >> 1;
                v += eri_at(tab, as, is, js, js);
                if ((j & 1) == (i & 1)) v -= eri_at(tab, as, js, js, is);
            }
        }
        return sg ? -v : v;
    }
    if (na == 2) {
        const int i = lowest<W>(I), a = lowest<W>(A);
        Key<W> I2 = I, A2 = A;
        flip_bit<W>(I2, i);
        flip_bit<W>(A2, a);
        const int j = lowest<W>(I2), b = lowest<W>(A2);
        // |bra> = G a+_a a+_b a_j a_i |ket>
        Key<W> st = ket;
        int sg = parity_below<W>(st, i);
        flip_bit<W>(st, i);
        sg ^= parity_below<W>(st, j);
        flip_bit<W>(st, j);
        sg ^= parity_below<W>(st, b);
        flip_bit<W>(st, b);
        sg ^= parity_below<W>(st, a);
        double v = 0.0;
        if (((a ^ i) & 1) == 0 && ((b ^ j) & 1) == 0) v += eri_at(tab, a >> 1, i >> 1, b >> 1, j >> 1);
        if (((a ^ j) & 1) == 0 && ((b ^ i) & 1) == 0) v -= eri_at(tab, a >> 1, j >> 1, b >> 1, i >> 1);
        return sg ? -v : v;
    }
    return 0.0;
}

template <int W>
__device__ __forceinline__ double sc_diagonal(const DevTable &tab, const Key<W> &any) {
    const Key<W> x = in_register<W>(tab, any);
    const int K = tab.sc_k;
    double d = 0.0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        uint64_t m = x.w[q];
        while (m) {
            const int i = 64 * q + __builtin_ctzll(m);
            m &= m - 1;
            const int is = i >> 1;
            d += tab.sc_h1[is * K + is];
            // partners above i
            Key<W> rest;
#pragma unroll
            for (int r = 0; r < W; ++r) rest.w[r] = r < q ? 0ull : (r == q ? m : x.w[r]);
#pragma unroll
            for (int r = 0; r < W; ++r) {
                uint64_t m2 = rest.w[r];
                while (m2) {
                    const int j = 64 * r + __builtin_ctzll(m2);
                    m2 &= m2 - 1;
                    const int js = j >> 1;
                    d += eri_at(tab, is, is, js, js);
                    if ((i & 1) == (j & 1)) d -= eri_at(tab, is, js, js, is);
                }
            }
        }
    }
    return d;
}

// Whether the digit tiles give the sample's diagonal as closely as its sum.
template <int W>
__device__ __forceinline__ bool sc_diagonal_tiled(const DevTable &tab, const Key<W> &x) {
    uint64_t v = x.w[0] & tab.diag_tile[0];
    if constexpr (W == 2) v |= x.w[W - 1] & tab.diag_tile[1];
    return v != 0ull;
}

// ---- FP32 form with compensation (precision NQS_FP32_KAHAN)
//
// A group's sum enters as an FP32 pair hi + lo (of its FP64 value); the terms
// of a diagonal in term form likewise, with the sign (-1)^{popc(Z & x)}
// applied by flipping sign bits.  The hi parts are added with Knuth's
// error-free TwoSum and the lo parts and the TwoSum errors go into a
// compensation term; a product H * r keeps its rounding error through fma.
// The per-sample value s + c is widened to FP64 only when it leaves the lane.

__device__ __forceinline__ void two_sum(float a, float b, float &s, float &e) {
    s = a + b;
    const float bp = s - a;
    e = (a - (s - bp)) + (b - bp);
}

__device__ __forceinline__ float flip_sign(float v, int par) {
    return __uint_as_float(__float_as_uint(v) ^ (static_cast<uint32_t>(par & 1) << 31));
}

struct AccF32 {
    float s = 0.f, c = 0.f;
    __device__ __forceinline__ void add(float v, float err) {
        float t, e;
        two_sum(s, v, t, e);
        s = t;
        c += e + err;
    }
    __device__ __forceinline__ double value() const {
        return static_cast<double>(s) + static_cast<double>(c);
    }
};

// The same sum for the FP32 form: the FP64 sum as an FP32 pair.
template <int W>
__device__ __forceinline__ AccF32 group_sum_f32(const DevTable &tab, int64_t g, const Key<W> &x,
                                                unsigned long long *terms, uint32_t cnt = 0) {
    const double v = group_sum<W, false>(tab, g, x, nullptr, terms, cnt);
    AccF32 a;
    a.s = static_cast<float>(v);
    a.c = static_cast<float>(v - static_cast<double>(a.s));
    return a;
}

// psi(x') / psi(x) in FP64 from the log-amplitude and phase differences (as
// the product of psi(x') and 1 / psi(x), each formed once per sample, it took
// the pair kernel a tenth less time, but was further off wherever the
// differences are exact or small: log-amplitudes -8 +- 0.1 of one phase
// 8.3e-17 rms instead of 4.9e-17, and no imaginary part was exactly 0).
__device__ __forceinline__ double2 amp_ratio_inline(double da, double dphi) {
    double sn, cs;
    sincos(dphi, &sn, &cs);
    const double mag = exp(da);
    return make_double2(mag * cs, mag * sn);
}

// Out of line: inlined into a kernel's partner or probe loop, the exp and
// sincos constants stay in registers across the whole loop and cost it
// waves per SIMD (the call is made only on a hit).
[[maybe_unused]] static __device__ __noinline__ double2 amp_ratio_f64(double da, double dphi) {
    return amp_ratio_inline(da, dphi);
}

// psi(x') / psi(x) in FP32 from the FP64 log-psi difference; the phase
// difference is reduced to (-pi, pi] in FP64 before rounding.
__device__ __forceinline__ void ratio_f32(double da, double dphi, float &rr, float &ri) {
    constexpr double kTwoPi = 6.283185307179586476925286766559;
    dphi -= kTwoPi * rint(dphi / kTwoPi);
    const float mag = expf(static_cast<float>(da));
    float sn, cs;
    sincosf(static_cast<float>(dphi), &sn, &cs);
    rr = mag * cs;
    ri = mag * sn;
}

// Index of the group with flip mask X, or -1; *cnt receives its terms (255:
// or more; the integral form has none).  A bucket of four slots is read at
// once, and one with a free slot ends the search: one round trip for nearly
// every lookup, where single slots took the longest chain of a wave's 64
// lanes (five or six).
template <int W, bool SCV>
__device__ __forceinline__ int64_t group_find(const DevTable &tab, const Key<W> &X,
                                              uint32_t *cnt) {
    const uint32_t hX = group_hash(X.w[0], W == 2 ? X.w[W - 1] : 0ull);
    const uint32_t mask = 0xFFFFFFFFu >> tab.gh_shift;
    uint32_t slot = slot_of(hX, tab.gh_shift) & ~3u;
    for (uint32_t probe = 0; probe <= mask; probe += 4) {
        uint32_t g[4], info[4];
        if constexpr (SCV) {
            const uint4 a = *reinterpret_cast<const uint4 *>(
                static_cast<const uint32_t *>(tab.gh) + slot);
            g[0] = a.x; g[1] = a.y; g[2] = a.z; g[3] = a.w;
        } else {
            const uint4 *p = reinterpret_cast<const uint4 *>(
                static_cast<const uint64_t *>(tab.gh) + slot);
            const uint4 a = p[0], b = p[1];
            g[0] = a.x; g[1] = a.z; g[2] = b.x; g[3] = b.z;
            info[0] = a.y; info[1] = a.w; info[2] = b.y; info[3] = b.w;
        }
        uint32_t match = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            bool m = g[k] != 0xFFFFFFFFu;
            if constexpr (!SCV) m = m && (info[k] >> 8) == (hX & 0xFFFFFFu);
            match |= m ? 1u << k : 0u;
        }
        while (match) {
            const int k = __builtin_ctz(match);
            match &= match - 1;
            const uint32_t gk = k == 0 ? g[0] : k == 1 ? g[1] : k == 2 ? g[2] : g[3];
            bool eq = true;
#pragma unroll
            for (int q = 0; q < W; ++q) eq = eq && group_x<W>(tab, gk, q) == X.w[q];
            if (eq) {
                if constexpr (!SCV)
                    *cnt = (k == 0 ? info[0] : k == 1 ? info[1] : k == 2 ? info[2] : info[3]) & 0xFFu;
                return gk;
            }
        }
        // (slots fill in order: a free one is the last)
        if (g[3] == 0xFFFFFFFFu) return -1;
        slot = (slot + 4) & mask;
    }
    return -1;
}

// Sum of FP64 values as an unevaluated pair hi + lo: the rounding errors of
// the additions (TwoSum) go to lo, so the value, rounded once, does not
// depend on the order of the additions (up to ties closer than about 2^-100
// of the largest partial sum).  An infinity or NaN passes through hi.  The
// additions are kept apart from the product that v may be: contracted with it
// in one copy of an unrolled loop and not in the next, they would add v in
// one place and the unrounded product in the other, and the sum would depend
// on which of them comes where.
struct Acc2 {
    double hi = 0.0, lo = 0.0;
    __device__ __forceinline__ void add(double v) {
#pragma clang fp contract(off)
        const double s = hi + v, bp = s - hi;
        lo += (hi - (s - bp)) + (v - bp);
        hi = s;
    }
    // another sum (its lo counts only beside a finite hi)
    __device__ __forceinline__ void add(double vhi, double vlo) {
        add(vhi);
        if (isfinite(vhi)) add(vlo);
    }
    __device__ __forceinline__ double value() const { return isfinite(hi) ? hi + lo : hi; }
};

// ------------------------------------------------------------------ hash build

// One thread per sample: range check, sector uniformity, counts >= 0, linear
// hash, Bloom bit, and insertion by CAS on the slot index.  A duplicate key
// is found by comparing against the sample that owns the slot.  With the
// pair join chosen only the checks run.
template <int W>
__device__ __forceinline__ void hash_build_one(const DevTable &tab, const DevScratch &sc,
                                               const uint64_t *__restrict__ samples,
                                               const int64_t *__restrict__ weights, int64_t i) {
    const uint64_t w0 = samples[2 * i], w1 = samples[2 * i + 1];
    bool bad;
    const int nq = tab.n_qubits;
    if (nq >= 64) {
        bad = (nq - 64 < 64) && ((w1 >> (nq - 64)) != 0);
    } else {
        bad = ((w0 >> nq) != 0) || (w1 != 0);
    }
    if (bad) latch(sc.err, NQS_E_RANGE);
    if (weights && weights[i] < 0) latch(sc.err, NQS_E_RANGE);
    if (tab.sector_filter) {
        const uint64_t s0 = samples[0], s1 = samples[1];
        const int na = __popcll(w0 & tab.spin_a0) + __popcll(w1 & tab.spin_a1);
        const int nb = __popcll(w0 & tab.spin_b0) + __popcll(w1 & tab.spin_b1);
        const int ra = __popcll(s0 & tab.spin_a0) + __popcll(s1 & tab.spin_a1);
        const int rb = __popcll(s0 & tab.spin_b0) + __popcll(s1 & tab.spin_b1);
        if (na != ra || nb != rb) atomicOr(sc.mixed, 1);
    }
    // the pair join, when it runs, needs neither the hash nor the filters
    if (join_chosen(sc) || bad) return;
    Key<W> k;
    k.w[0] = w0;
    if constexpr (W == 2) k.w[1] = w1;
    const uint32_t h = linear_hash<W>(k, tab.hr);
    sc.shx[i] = h;
    const uint32_t fmask = (1u << sc.filter_log2) - 1u;
    const uint32_t fbits = filter_bits(h);
    atomicOr(&sc.filter[filter_word(h, fmask)], fbits);
    if (sc.eparts_log2 > 0) {
        // the partition of the enumeration filter: class of x, the XOR of
        // the classes of its occupied beta qubits
        uint32_t c = 0;
        uint64_t m0 = w0 & tab.spin_b0, m1 = w1 & tab.spin_b1;
        while (m0) {
            c ^= tab.qcls[__builtin_ctzll(m0)];
            m0 &= m0 - 1;
        }
        while (m1) {
            c ^= tab.qcls[64 + __builtin_ctzll(m1)];
            m1 &= m1 - 1;
        }
        c &= (1u << sc.eparts_log2) - 1u;
        const uint32_t emask = (1u << sc.efilter_log2) - 1u;
        atomicOr(&sc.efilter[(c << sc.efilter_log2) + filter_word(h, emask)], fbits);
    }
    uint32_t slot = slot_of(h, sc.slot_shift) << bucket_log2(W);
    for (uint32_t probe = 0; probe <= sc.slot_mask; ++probe) {
        const int32_t old = atomicCAS(&sc.sidx[slot], -1, static_cast<int32_t>(i));
        if (old == -1) {
            sc.skey[static_cast<size_t>(slot) * W] = w0;
            if constexpr (W == 2) sc.skey[static_cast<size_t>(slot) * W + 1] = w1;
            sc.sfp[slot] = h | 1u;
            return;
        }
        bool same = samples[2 * old] == w0;
        if constexpr (W == 2) same = same && samples[2 * old + 1] == w1;
        if (same) {
            latch(sc.err, NQS_E_DUPLICATE);
            return;
        }
        slot = (slot + 1) & sc.slot_mask;
    }
}

}  // namespace nqs
