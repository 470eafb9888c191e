// Span passes: Pauli rotations on tiles that are cosets of a subspace of the
// index space (see span.cpp), gfx950.
//
// A workgroup of 2^LOGT threads holds a tile of 2^(LOGT + LR) amplitudes in
// registers, 2^LR per thread.  In every stage the rotations' X masks are single
// bits of the register index (or none), so a rotation
//     y[i] = a (x[i] + t (-1)^(i . z) x[i ^ x])
// is arithmetic between a thread's own registers: two multiply-adds an
// amplitude, t = +-tan phi real or imaginary, the cosine a taken out into the
// scale of the pass.  The sign is linear in the index: one parity for the tile, one per
// thread, one bit per register.  Between stages the tile goes through LDS: a
// thread writes its registers to the slots of the old layout and reads those
// of the new one.  It reads and later rewrites the same slots, so one barrier
// per re-layout is enough.
//
// What bounds it: the trip of the tile through memory, then what of the
// rotations the other workgroups of a CU do not hide.  At 21 qubits two
// workgroups a CU hold every tile and do the same at the same time, so that the
// parts add up: complex128 17.5 us a pass, of which a copy whose blocks change
// XCD takes 11.3, vector instructions 3.3 and the LDS 2.0; complex64 15.4 of 7.8,
// 3.8 and 1.1 (counters of 11 rotations a pass).  At 30 qubits a pass is 88% of
// the rate of a copy.  So the work around a rotation's 32 multiply-adds is kept
// small: an entry of 16 bytes per rotation (one LDS read, two words moved to
// scalar registers), the tile's sign joined to t beforehand, eight sign changes in
// place, byte offsets in 32 bits where they fit, the scale multiplied once per
// pass.  Against records and coefficients decoded per rotation, us per pass:
// 21 qubits complex128 19.4 -> 17.5, complex64 16.7 -> 15.4, 24 qubits complex128
// 120 -> 114, 30 qubits complex64 3681 -> 3626 to 3710 on several machines.
// Plain loads and stores: non-temporal ones, which suit k_tile's passes, cost
// 1540 us against 925 per pass at 27 qubits complex128 and 5174 against 3681 at
// 30 qubits complex64 (22.1 against 19.4 at 21 qubits complex128).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "device.h"
#include "launch.h"

namespace qk {

using qs::DevOp;

// v with its sign flipped where bit 31 of s (no other bit set) is
__device__ __forceinline__ float flip(float v, uint32_t s) { return __uint_as_float(__float_as_uint(v) ^ s); }
__device__ __forceinline__ double flip(double v, uint32_t s) {
    return __longlong_as_double(__double_as_longlong(v) ^ (int64_t(uint64_t(s) << 32)));
}
// The same in place, for a sign that is the same on every lane: one operation.
// (Left to itself the compiler copies the other half of a double each time.)
__device__ __forceinline__ void turn(float &v, uint32_t s) {
    uint32_t u = __float_as_uint(v);
    asm("v_xor_b32 %0, %1, %0" : "+v"(u) : "s"(s));
    v = __uint_as_float(u);
}
__device__ __forceinline__ void turn(double &v, uint32_t s) {
    typedef uint32_t U2 __attribute__((ext_vector_type(2)));
    U2 u = __builtin_bit_cast(U2, v);
    uint32_t hi = u.y;
    asm("v_xor_b32 %0, %1, %0" : "+v"(hi) : "s"(s));
    u.y = hi;
    v = __builtin_bit_cast(double, u);
}

// XOR of the register bits' vectors over the bits of R
template <int R, typename V>
__device__ __forceinline__ V reg_off(const V *vec) {
    V o = 0;
    static_for<0, qs::kSpanRegs>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if constexpr ((R >> k) & 1) o ^= vec[k];
    });
    return o;
}

// Register r of place g in an order of the register index in which neighbours
// differ in one bit, M left out (its bit 0): a Gray code of the other bits.
template <int M>
__device__ constexpr int gray_reg(int g) {
    const int c = g ^ (g >> 1);
    return M == 0 ? c : (c / M) * (2 * M) + c % M;
}

// The signs of the register bits, from the low bits of a record's word: s[b] has
// bit 31 set where bit b's sign mask is.
template <int LR>
struct Signs {
    uint32_t s[LR];
    __device__ __forceinline__ explicit Signs(uint32_t w) {
        static_for<0, LR>([&](auto bc) {
            constexpr int b = decltype(bc)::value;
            s[b] = (w << (31 - b)) & 0x80000000u;
        });
    }
};

// One rotation from a thread's registers x to y, y[r] = x[r] + t_r x[r ^ M] with
// M one register bit or none, t real (REAL) or imaginary.  t has the sign of
// register 0 (and of the tile and the thread).  The pairs {r, r ^ M} follow in
// Gray code order, so that the next pair's sign is one operation away, with one
// of few scalars.  Register r ^ M has the sign of r for an imaginary t (an even
// number of Y letters) and the opposite one for a real t.
template <typename T, int LR, int M, bool REAL>
__device__ __forceinline__ void rotate(const Cx<T> (&x)[1 << LR], Cx<T> (&y)[1 << LR], T t, uint32_t w) {
    const Signs<LR> sg(w);
    static_for<0, (M == 0 ? 1 << LR : 1 << (LR - 1))>([&](auto gc) {
        constexpr int g = decltype(gc)::value, r = gray_reg<M>(g), q = r ^ M;
        if constexpr (g > 0) turn(t, sg.s[__builtin_ctz(r ^ gray_reg<M>(g - 1))]);
        const Cx<T> a = x[r], b = x[q];
        if constexpr (REAL) {
            y[r] = Cx<T>{T(fma(t, b.re, a.re)), T(fma(t, b.im, a.im))};
            y[q] = Cx<T>{T(fma(-t, a.re, b.re)), T(fma(-t, a.im, b.im))};
        } else {
            y[r] = Cx<T>{T(fma(-t, b.im, a.re)), T(fma(t, b.re, a.im))};
            if constexpr (M != 0) y[q] = Cx<T>{T(fma(-t, a.im, b.re)), T(fma(t, a.re, b.im))};
        }
    });
    // Differs from form to form: the compiler would else merge the tails of
    // the switch over them, whose register operands it then has to address.
    asm volatile("; rotated by %0" ::"i"(M * 2 + REAL));
}

// form: 2 b + REAL for register bit b, 2 LR for no register bit (a diagonal)
template <typename T, int LR>
__device__ __forceinline__ void rotate_form(const Cx<T> (&x)[1 << LR], Cx<T> (&y)[1 << LR], int form, T t, uint32_t d) {
    static_assert(LR == 4, "forms of four register bits");
    switch (form) {
    case 0: rotate<T, LR, 1, false>(x, y, t, d); break;
    case 1: rotate<T, LR, 1, true>(x, y, t, d); break;
    case 2: rotate<T, LR, 2, false>(x, y, t, d); break;
    case 3: rotate<T, LR, 2, true>(x, y, t, d); break;
    case 4: rotate<T, LR, 4, false>(x, y, t, d); break;
    case 5: rotate<T, LR, 4, true>(x, y, t, d); break;
    case 6: rotate<T, LR, 8, false>(x, y, t, d); break;
    case 7: rotate<T, LR, 8, true>(x, y, t, d); break;
    default: rotate<T, LR, 0, false>(x, y, t, d); break;
    }
}

// The bits in which two numbers differ, and the change from one to the other where
// m is all ones (0: none): one operation a word.
struct Bits1 {
    uint32_t lo;
};
struct Bits2 {
    uint32_t lo, hi;
};
__device__ __forceinline__ Bits1 differ(float u, float v) { return {__float_as_uint(u) ^ __float_as_uint(v)}; }
__device__ __forceinline__ Bits2 differ(double u, double v) {
    const uint64_t d = uint64_t(__double_as_longlong(u) ^ __double_as_longlong(v));
    return {uint32_t(d), uint32_t(d >> 32)};
}
__device__ __forceinline__ void change(float &u, Bits1 d, uint32_t m) { u = __uint_as_float(__float_as_uint(u) ^ (d.lo & m)); }
__device__ __forceinline__ void change(double &u, Bits2 d, uint32_t m) {
    const uint64_t b = uint64_t(__double_as_longlong(u));
    u = __longlong_as_double(int64_t(uint64_t(uint32_t(b) ^ (d.lo & m)) | (uint64_t(uint32_t(b >> 32) ^ (d.hi & m)) << 32)));
}

// A rotation of two angles: as rotate, but y[r] = a x[r] + b x[r ^ M] in full, with
// (a, b) that of the branch of register r: register 0's is (a, b), the other differs
// by (da, db), and the branch changes with the parity of r and bits 4-7 of w, which
// leave out M.  Where an angle is 0 the amplitudes stay as they are to the last bit,
// and none of it goes into the pass's scale.
template <typename T, int LR, int M, bool REAL, typename D>
__device__ __forceinline__ void rotate2(const Cx<T> (&x)[1 << LR], Cx<T> (&y)[1 << LR], T a, T b, D da, D db, uint32_t w) {
    const Signs<LR> sg(w);
    static_for<0, (1 << (LR - 1))>([&](auto gc) {
        constexpr int g = decltype(gc)::value, r = gray_reg<M>(g), q = r ^ M;
        if constexpr (g > 0) {
            constexpr int bit = __builtin_ctz(r ^ gray_reg<M>(g - 1));
            const uint32_t m = uint32_t(int32_t(w << (31 - LR - bit)) >> 31);
            turn(b, sg.s[bit]);
            change(a, da, m);
            change(b, db, m);
        }
        const Cx<T> u = x[r], v = x[q];
        if constexpr (REAL) {
            y[r] = Cx<T>{T(fma(b, v.re, a * u.re)), T(fma(b, v.im, a * u.im))};
            y[q] = Cx<T>{T(fma(-b, u.re, a * v.re)), T(fma(-b, u.im, a * v.im))};
        } else {
            y[r] = Cx<T>{T(fma(-b, v.im, a * u.re)), T(fma(b, v.re, a * u.im))};
            y[q] = Cx<T>{T(fma(-b, u.im, a * v.re)), T(fma(b, u.re, a * v.im))};
        }
    });
    asm volatile("; turned by %0" ::"i"(M * 2 + REAL));   // (as in rotate)
}

template <typename T, int LR, typename D>
__device__ __forceinline__ void rotate2_form(const Cx<T> (&x)[1 << LR], Cx<T> (&y)[1 << LR], int form, T a, T b, D da,
                                             D db, uint32_t w) {
    switch (form) {
    case 0: rotate2<T, LR, 1, false>(x, y, a, b, da, db, w); break;
    case 1: rotate2<T, LR, 1, true>(x, y, a, b, da, db, w); break;
    case 2: rotate2<T, LR, 2, false>(x, y, a, b, da, db, w); break;
    case 3: rotate2<T, LR, 2, true>(x, y, a, b, da, db, w); break;
    case 4: rotate2<T, LR, 4, false>(x, y, a, b, da, db, w); break;
    case 5: rotate2<T, LR, 4, true>(x, y, a, b, da, db, w); break;
    case 6: rotate2<T, LR, 8, false>(x, y, a, b, da, db, w); break;
    default: rotate2<T, LR, 8, true>(x, y, a, b, da, db, w); break;
    }
}

// LDS behind the tile: an entry of 16 bytes per record, the layouts of the
// stages (64 bytes each) and a factor of the pass's scale per record.
typedef uint32_t U4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) U4 LdsU4;
typedef __attribute__((address_space(3))) double LdsF8;

// An entry.  Word 0: the form (bits 28-31; kStageForm: a stage, its number in
// the low bits), the sign masks of the thread (bits 16-27) and of the register
// index (bits 0-3).  Word 1: not 0 where the scale so far is to be applied.  t: the upper
// half (complex128) or word 2.
// A measurement record: form kRecForm, its masks, dimension and value as in the
// device record (bits 16-27, 0-7), its kind (bits 8-11), its slot in word 1 and
// the layout of a failing state in word 2.
// A rotation of two angles: form kPairForm, the sign masks of the thread and of
// the register index as above, the branch's masks in word 1 (thread) and bits
// 4-7, the form of rotate2_form in bits 8-10; the next two entries hold the
// cosine and sine of the branch of thread 0's register 0, and of the other (both
// in the first of them in single precision).
constexpr uint32_t kStageForm = 15, kRecForm = 14, kPairForm = 13;
__device__ __forceinline__ void put_t(U4 &e, float t) { e.z = __float_as_uint(t); }
__device__ __forceinline__ void put_t(U4 &e, double t) {
    const uint64_t b = uint64_t(__double_as_longlong(t));
    e.z = uint32_t(b);
    e.w = uint32_t(b >> 32);
}
template <typename T>
__device__ __forceinline__ T get_t(const U4 &e) {
    if constexpr (sizeof(T) == 4) return __uint_as_float(e.z);
    else return __longlong_as_double(int64_t(uint64_t(e.z) | (uint64_t(e.w) << 32)));
}
__device__ __forceinline__ U4 lds_u4(uint32_t at) { return *reinterpret_cast<const LdsU4 *>(uintptr_t(at)); }

// A layout in LDS: the byte address that each position adds, 32 bits each, from
// the 16-bit slots of a stage record (words a and c).
constexpr uint32_t kLayoutBytes = 64;
template <typename T>
__device__ __forceinline__ void put_layout(uint32_t at, const U4 &a, const U4 &c) {
    constexpr int LOGE = LdsTile<T>::LOGE;
    auto lo = [](uint32_t w) { return (w & 0xffffu) << LOGE; };
    auto hi = [](uint32_t w) { return (w >> 16) << LOGE; };
    const U4 q[4] = {{lo(a.x), hi(a.x), lo(a.y), hi(a.y)},
                     {lo(a.z), hi(a.z), lo(a.w), lo(c.x)},
                     {hi(c.x), lo(c.y), hi(c.y), lo(c.z)},
                     {hi(c.z), lo(c.w), 0u, hi(c.w)}};
#pragma unroll
    for (int j = 0; j < 4; j++) *reinterpret_cast<LdsU4 *>(uintptr_t(at + 16u * j)) = q[j];
}

// The byte addresses of a thread's elements under the layout at `at`.
template <typename T, int LOGT>
__device__ __forceinline__ void stage_addr(uint32_t at, int tid, uint32_t (&addr)[1 << qs::kSpanRegs]) {
    constexpr int LR = qs::kSpanRegs;
    uint32_t h[16];
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const U4 q = lds_u4(at + 16u * j);
        h[4 * j] = q.x;
        h[4 * j + 1] = q.y;
        h[4 * j + 2] = q.z;
        h[4 * j + 3] = q.w;
    }
    uint32_t a = h[15];   // (0 but for the layout of a failing state)
    static_for<0, LOGT>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        a ^= ((tid >> k) & 1) ? h[k] : 0;
    });
    addr[0] = a;
    static_for<1, 1 << LR>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        addr[r] = addr[r & (r - 1)] ^ h[LOGT + __builtin_ctz(r)];
    });
}

template <bool WIDE>
struct OffsetOf {
    typedef uint32_t type;
};
template <>
struct OffsetOf<true> {
    typedef uint64_t type;
};

// Sum over a wave, in lane 63 (fixed order; row shifts and row broadcasts, no LDS).
__device__ __forceinline__ double wave_total(double v) {
    auto step = [&](auto ctrl, auto rows) {
        const int64_t b = __double_as_longlong(v);
        const int lo = __builtin_amdgcn_update_dpp(0, int(uint32_t(b)), decltype(ctrl)::value, decltype(rows)::value, 0xf, true);
        const int hi = __builtin_amdgcn_update_dpp(0, int(b >> 32), decltype(ctrl)::value, decltype(rows)::value, 0xf, true);
        v += __longlong_as_double((int64_t(hi) << 32) | int64_t(uint32_t(lo)));
    };
    step(IntC<0x111>{}, IntC<0xf>{});   // row_shr 1, 2, 4, 8: lane 15 of a row holds its sum
    step(IntC<0x112>{}, IntC<0xf>{});
    step(IntC<0x114>{}, IntC<0xf>{});
    step(IntC<0x118>{}, IntC<0xf>{});
    step(IntC<0x142>{}, IntC<0xa>{});   // row_bcast 15 into rows 1 and 3, 31 into rows 2 and 3
    step(IntC<0x143>{}, IntC<0xc>{});
    return v;
}

// A measurement record on a tile that is the whole state: the weights of both
// values in FP64 (each thread's in order, its wave's, the waves' in order), the
// decision as in k_tile's records, and the collapse.  Returns 0 or a negative
// status, the registers then untouched.  *collapsed: the state was scaled to
// norm 1, `sign` being that of the scale that the rotations before left out.
template <typename T, int LOGT>
__device__ __forceinline__ int span_record(Cx<T> (&v)[1 << qs::kSpanRegs], uint32_t w, uint32_t slot, int tid,
                                           uint32_t red_at, double sign, const MeasArgs &ma, uint32_t b,
                                           bool *collapsed) {
    constexpr int E = 1 << qs::kSpanRegs, NW = (1 << LOGT) / 64;
    const uint32_t fr = w & 15u, dir = (w >> 4) & 7u;
    const int kind = int((w >> 8) & 15u);
    const bool tb = ((__builtin_popcount(uint32_t(tid) & ((w >> 16) & 0xfffu)) + int((w >> 7) & 1u)) & 1) != 0;
    auto reg_bit = [&](int r) { return ((0x6996u >> (uint32_t(r) & fr)) & 1u) != 0; };
    double w0 = 0.0, w1 = 0.0;
    static_for<0, E>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        const double re = double(v[r].re), im = double(v[r].im), n2 = re * re + im * im;
        w0 += reg_bit(r) ? 0.0 : n2;
        w1 += reg_bit(r) ? n2 : 0.0;
    });
    const double a0 = wave_total(tb ? w1 : w0), a1 = wave_total(tb ? w0 : w1);
    if ((tid & 63) == 63) {
        *reinterpret_cast<LdsF8 *>(uintptr_t(red_at + 16u * uint32_t(tid >> 6))) = a0;
        *reinterpret_cast<LdsF8 *>(uintptr_t(red_at + 16u * uint32_t(tid >> 6) + 8u)) = a1;
    }
    __syncthreads();
    double P0 = 0.0, P1 = 0.0;
    for (int j = 0; j < NW; j++) {
        P0 += *reinterpret_cast<const LdsF8 *>(uintptr_t(red_at + 16u * uint32_t(j)));
        P1 += *reinterpret_cast<const LdsF8 *>(uintptr_t(red_at + 16u * uint32_t(j) + 8u));
    }
    __syncthreads();   // the next record may write the scratch
    // registers exchanged along the direction that flips the value
    auto move = [&]() {
        auto along = [&](auto mc) {
            constexpr int M = decltype(mc)::value;
            static_for<0, E>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                if constexpr (!(r & M)) {
                    const Cx<T> a = v[r];
                    v[r] = v[r | M];
                    v[r | M] = a;
                }
            });
            asm volatile("; moved along %0" ::"i"(M));   // (as in rotate)
        };
        if (dir == 1) along(IntC<1>{});
        else if (dir == 2) along(IntC<2>{});
        else if (dir == 3) along(IntC<4>{});
        else along(IntC<8>{});
    };
    if (kind == qs::DEVOP_RESET) {
        if (P1 == 0.0) return 0;
        if (P0 != 0.0) return QSIM_E_NOT_DEFINITE;
        move();
        return 0;
    }
    int o;
    const size_t idx = size_t(b) * ma.nslots + slot;
    if (kind == qs::DEVOP_ASSERT0) {
        if (!(P0 > 0.0)) return QSIM_E_ZERO_PROB;
        o = 0;
    } else if (ma.forced && ma.forced[idx] >= 0) {
        o = ma.forced[idx];
        if (!((o ? P1 : P0) > 0.0)) return QSIM_E_ZERO_PROB;
    } else {
        o = ma.uniforms[idx] < P0 / (P0 + P1) ? 0 : 1;
    }
    o = __builtin_amdgcn_readfirstlane(o);
    const double kept = o ? P1 : P0;
    if (tid == 0) {
        ma.outcomes[idx] = o;
        ma.probs[idx] = kept / (P0 + P1);
    }
    const T f = T((sign < 0.0 ? -1.0 : 1.0) / sqrt(kept));
    static_for<0, E>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        const bool keep = (tb != reg_bit(r)) == (o != 0);
        v[r] = keep ? Cx<T>{v[r].re * f, v[r].im * f} : Cx<T>{T(0), T(0)};
    });
    if (kind == qs::DEVOP_MEASURE_RESET && o) move();
    *collapsed = true;
    return 0;
}

// WIDE: byte offsets inside a state need more than 32 bits.  MEAS: the pass holds
// measurement records.  PAIR: it holds rotations of two angles (a kernel of its
// own: their registers and branches would cost every other pass).
template <typename T, int LOGT, bool WIDE, bool MEAS, bool PAIR>
__global__ void __launch_bounds__(1 << LOGT) k_span(Cx<T> *__restrict__ state, uint64_t sstride, SpanArgs sa,
                                                   const DevOp *__restrict__ ops, uint32_t ob, uint32_t oe,
                                                   const Cx<T> *__restrict__ coefs, uint32_t cb, uint64_t cstride,
                                                   MeasArgs ma, uint32_t flags) {
    using L = LdsTile<T>;
    using Off = typename OffsetOf<WIDE>::type;
    constexpr int LR = qs::kSpanRegs, E = 1 << LR, TNT = 1 << LOGT;
    const uint32_t b = blockIdx.y;
    if (ma.status && ma.status[b] != 0) return;   // an earlier step of this state failed
    char *st = reinterpret_cast<char *>(state + size_t(b) * sstride);
    const Cx<T> *gcf = coefs + size_t(b) * cstride + cb;
    const int tid = threadIdx.x;
    const uint32_t nrec = oe - ob;
    const uint32_t ent_at = sa.tile_bytes, lay_at = ent_at + 16u * (nrec + 1), fac_at = lay_at + kLayoutBytes * sa.nlayout;
    const uint32_t red_at = fac_at + 8u * nrec, nrun = sa.nrun;
    const uint64_t base = span_base(blockIdx.x, sa);
    // byte offset of a thread's register 0, and what each register bit changes
    auto offsets = [&](const uint64_t *vec, Off (&reg)[LR]) {
        Off off = Off(base) << L::LOGE;
        static_for<0, LOGT>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            off ^= ((tid >> k) & 1) ? Off(vec[k]) << L::LOGE : Off(0);
        });
        static_for<0, LR>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            reg[k] = Off(vec[LOGT + k]) << L::LOGE;
        });
        return off;
    };

    Cx<T> v[E];
    {
        Off reg[LR];
        const Off off = offsets(sa.load_v, reg);
        if (flags & TF_INIT_ZERO) {
            static_for<0, E>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                v[r] = Cx<T>{T((off ^ reg_off<r>(reg)) == 0 ? 1 : 0), T(0)};
            });
        } else {
            static_for<0, E>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                v[r] = *reinterpret_cast<const Cx<T> *>(st + (off ^ reg_off<r>(reg)));
            });
        }
    }
    // While the tile loads fly, one thread per record writes its entry: the
    // sign of the tile's base index joins t here, once per tile and rotation.
    for (uint32_t x = uint32_t(tid); x < nrec; x += TNT) {
        const U4 *p = reinterpret_cast<const U4 *>(ops + ob + x);
        // (every record has two coefficients, so that they need not wait for it)
        const U4 a = p[0], c = p[1];
        const Cx<T> e0 = gcf[2 * x], e1 = gcf[2 * x + 1];
        U4 e = {0, 0, 0, 0};
        double f = 1.0;
        if (((a.w >> 16) & 0xff) == qs::DEVOP_PAULI) {
            const uint64_t zb = uint64_t((c.x >> 16) | (c.y << 16)) | (uint64_t(c.y >> 16) << 32);
            e.x = (a.y & 0xfu) | ((c.x & 0xfffu) << 16) | ((a.z & 0xffu) << 28);
            e.y = e1.re != T(0);
            put_t(e, flip(e1.im, uint32_t(__builtin_popcountll(base & zb)) << 31));
            f = double(e0.re) + double(e0.im);
        } else if (PAIR && ((a.w >> 16) & 0xff) == qs::DEVOP_PAULI2) {
            // the signs and the branch of the tile's base index join the coefficients
            const U4 a1 = p[2], c1 = p[3];
            const uint64_t zb = uint64_t((c.x >> 16) | (c.y << 16)) | (uint64_t(c.y >> 16) << 32);
            const uint64_t wb = uint64_t((c1.x >> 16) | (c1.y << 16)) | (uint64_t(c1.y >> 16) << 32);
            const uint32_t s = uint32_t(__builtin_popcountll(base & zb)) << 31;
            const bool other = (__builtin_popcountll(base & wb) & 1) != 0;
            const Cx<T> u = other ? e1 : e0, o = other ? e0 : e1;
            e.x = (kPairForm << 28) | ((c.x & 0xfffu) << 16) | ((a.z & 7u) << 8) | ((a1.y & 0xfu) << 4) | (a.y & 0xfu);
            e.y = c1.x & 0xfffu;
            if constexpr (sizeof(T) == 4) {
                const U4 d = {__float_as_uint(u.re), __float_as_uint(flip(u.im, s)), __float_as_uint(o.re),
                              __float_as_uint(flip(o.im, s))};
                *reinterpret_cast<LdsU4 *>(uintptr_t(ent_at + 16u * (x + 1))) = d;
            } else {
                auto words = [](double re, double im) {
                    const uint64_t r = uint64_t(__double_as_longlong(re)), i = uint64_t(__double_as_longlong(im));
                    return U4{uint32_t(r), uint32_t(r >> 32), uint32_t(i), uint32_t(i >> 32)};
                };
                *reinterpret_cast<LdsU4 *>(uintptr_t(ent_at + 16u * (x + 1))) = words(u.re, flip(u.im, s));
                *reinterpret_cast<LdsU4 *>(uintptr_t(ent_at + 16u * (x + 2))) = words(o.re, flip(o.im, s));
            }
        } else if (PAIR && ((a.w >> 16) & 0xff) == qs::DEVOP_PAULI2X) {
            *reinterpret_cast<LdsF8 *>(uintptr_t(fac_at + 8u * x)) = 1.0;
            continue;   // (its entry is written with the one before)
        } else if (MEAS && ((a.w >> 16) & 0xff) == qs::DEVOP_SPAN_REC) {
            e.x = (kRecForm << 28) | ((c.x & 0xfffu) << 16) | (((a.z >> 8) & 0xfu) << 8) | (a.y & 0xffu);
            e.y = (c.x >> 16) | (c.y << 16);
            e.z = a.w >> 24;
        } else {
            const uint32_t number = a.w >> 24;
            e.x = (kStageForm << 28) | number;
            put_layout<T>(lay_at + kLayoutBytes * number, a, c);
        }
        *reinterpret_cast<LdsU4 *>(uintptr_t(ent_at + 16u * x)) = e;
        *reinterpret_cast<LdsF8 *>(uintptr_t(fac_at + 8u * x)) = f;
    }
    __syncthreads();

    // the scale of records [lo, hi): lanes multiply the factors of theirs, then
    // each other's
    auto scale_of = [&](uint32_t lo, uint32_t hi) {
        double s = 1.0;
        for (uint32_t x = lo + (uint32_t(tid) & 63u); x < hi; x += 64u) {
            s *= *reinterpret_cast<const LdsF8 *>(uintptr_t(fac_at + 8u * x));
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) s *= __shfl_xor(s, d, 64);
        return s;
    };
    uint32_t addr[E];
    stage_addr<T, LOGT>(lay_at, tid, addr);
    // the next entry, and in single precision the one behind it, where a rotation of
    // two angles has its coefficients (in double precision the registers are short:
    // 12 qubits, 6 rounds, 222 us with those read ahead, 210 without; complex64 at 14
    // qubits, 8 rounds, 701 and 720).  LDS has room beyond the last entry.
    constexpr bool AHEAD2 = PAIR && sizeof(T) == 4;
    U4 ahead, ahead1 = {0, 0, 0, 0};
    auto read_ahead = [&](uint32_t i) __attribute__((always_inline)) {
        ahead = lds_u4(ent_at + 16u * i);
        if (AHEAD2) ahead1 = lds_u4(ent_at + 16u * (i + 1));
    };
    read_ahead(1);
    uint32_t scaled = 0;   // the first record whose factor the state does not have yet
    int failed = 0;
    // One record (with those behind it that belong to it: returns how many), from
    // the registers x to y.  (Two sets of registers in turn:
    // a rotation reads both members of a pair for both results, and in one set
    // every second result would have to be moved.)
    auto step = [&](uint32_t i, const Cx<T> (&x)[E], Cx<T> (&y)[E]) __attribute__((always_inline)) -> uint32_t {
        const U4 e = ahead;
        U4 d = ahead1;
        const uint32_t w = __builtin_amdgcn_readfirstlane(e.x);
        if (!AHEAD2) read_ahead(i + 1);
        const uint32_t form = w >> 28;
        if (AHEAD2) read_ahead(i + (form == kPairForm ? 3u : 1u));
        if (MEAS && form == kRecForm) {
            static_for<0, E>([&](auto rc) { y[decltype(rc)::value] = x[decltype(rc)::value]; });
            bool collapsed = false;
            failed = span_record<T, LOGT>(y, w, __builtin_amdgcn_readfirstlane(e.y), tid, red_at,
                                          scale_of(scaled, i), ma, b, &collapsed);
            failed = __builtin_amdgcn_readfirstlane(failed);
            if (collapsed) scaled = i + 1;
            if (failed) {
                // the state stays as it was before the record, in the order that
                // the frame had there
                if (tid == 0) {
                    ma.status[b] = failed;
                    if (ma.fail_at) ma.fail_at[b] = int(ob + i);
                }
                stage_addr<T, LOGT>(lay_at + kLayoutBytes * __builtin_amdgcn_readfirstlane(e.z), tid, addr);
            }
        } else if (PAIR && form == kPairForm) {
            U4 d2 = {0, 0, 0, 0};
            if (!AHEAD2) {
                d = ahead;
                d2 = lds_u4(ent_at + 16u * (i + 2));
                read_ahead(i + 3);
            }
            T a0, b0, a1, b1;
            if constexpr (sizeof(T) == 4) {
                a0 = __uint_as_float(d.x), b0 = __uint_as_float(d.y);
                a1 = __uint_as_float(d.z), b1 = __uint_as_float(d.w);
            } else {
                auto wide = [](uint32_t lo, uint32_t hi) { return __longlong_as_double(int64_t(uint64_t(lo) | (uint64_t(hi) << 32))); };
                a0 = wide(d.x, d.y), b0 = wide(d.z, d.w);
                a1 = wide(d2.x, d2.y), b1 = wide(d2.z, d2.w);
            }
            const uint32_t s = uint32_t(__builtin_popcount(uint32_t(tid) & ((w >> 16) & 0xfffu))) << 31;
            const bool other = (__builtin_popcount(uint32_t(tid) & e.y) & 1) != 0;
            rotate2_form<T, LR>(x, y, int((w >> 8) & 7u), other ? a1 : a0, flip(other ? b1 : b0, s), differ(a0, a1),
                                differ(b0, b1), w);
            return 3;
        } else if (form != kStageForm) {
            const uint32_t s = uint32_t(__builtin_popcount(uint32_t(tid) & ((w >> 16) & 0xfffu))) << 31;
            rotate_form<T, LR>(x, y, int(form), flip(get_t<T>(e), s), w);
            if (__builtin_amdgcn_readfirstlane(e.y)) {
                const T f = T(scale_of(scaled, i + 1));
                scaled = i + 1;
                static_for<0, E>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    y[r].re *= f;
                    y[r].im *= f;
                });
            }
        } else {
            // a stage: through LDS into its layout
            static_for<0, E>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                L::st(addr[r], x[r]);
            });
            stage_addr<T, LOGT>(lay_at + kLayoutBytes * (w & 0xffu), tid, addr);
            __syncthreads();
            static_for<0, E>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                y[r] = L::ld(addr[r]);
            });
        }
        return 1;
    };
    // (two steps a turn, between the two sets; a loop that leaves in the middle runs
    // 9-20% longer)
    const uint32_t nstep = PAIR ? nrun - 2 * sa.pairs : nrun;
    uint32_t i = 1, c = 1;   // record, step
    for (; c + 1 < nstep; c += 2) {
        Cx<T> u[E];
        uint32_t used = step(i, v, u);
        if (MEAS && failed) {
            static_for<0, E>([&](auto rc) { v[decltype(rc)::value] = u[decltype(rc)::value]; });
            break;
        }
        i += used;
        used = step(i, u, v);
        if (MEAS && failed) break;
        i += used;
    }
    if (c < nstep && !failed) {
        Cx<T> u[E];
        const uint32_t used = step(i, v, u);
        static_for<0, E>([&](auto rc) { v[decltype(rc)::value] = u[decltype(rc)::value]; });
        if (!(MEAS && failed)) i += used;
    }
    const double scale = scale_of(scaled, MEAS && failed ? i : nrun);
    const T fr = T(scale * sa.phase_re), fi = T(scale * sa.phase_im);
    const bool turned = sa.phase_im != 0.0;
    auto result = [&](const Cx<T> a) {
        Cx<T> y{a.re * fr, a.im * fr};
        if (turned) {
            y.re = fma(-fi, a.im, y.re);
            y.im = fma(fi, a.re, y.im);
        }
        return y;
    };
    if (MEAS && failed) {
        static_for<0, E>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            *reinterpret_cast<Cx<T> *>(st + addr[r]) = result(v[r]);
        });
    } else {
        Off reg[LR];
        const Off off = offsets(sa.store_v, reg) ^ (Off(sa.store_base) << L::LOGE);
        static_for<0, E>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            *reinterpret_cast<Cx<T> *>(st + (off ^ reg_off<r>(reg))) = result(v[r]);
        });
    }
}

// ---------------------------------------------------------- Pauli sums
// A term's sum over a thread's registers (see rotate for M, REAL and w): the
// real parts of conj(v[r]) v[r ^ M] with their signs, the imaginary parts for
// an odd number of Y letters (REAL), |v[r]|^2 for M = 0.
template <typename T, int LR, int M, bool REAL>
__device__ __forceinline__ double term_sum(const Cx<T> (&v)[1 << LR], double one, uint32_t w) {
    const Signs<LR> sg(w);
    double acc = 0.0;
    static_for<0, (M == 0 ? 1 << LR : 1 << (LR - 1))>([&](auto gc) {
        constexpr int g = decltype(gc)::value, r = gray_reg<M>(g), q = r ^ M;
        if constexpr (g > 0) turn(one, sg.s[__builtin_ctz(r ^ gray_reg<M>(g - 1))]);
        const double ar = v[r].re, ai = v[r].im, br = v[q].re, bi = v[q].im;
        acc = fma(one, REAL ? fma(ar, bi, -(ai * br)) : fma(ar, br, ai * bi), acc);
    });
    asm volatile("; summed by %0" ::"i"(M * 2 + REAL));
    return acc;
}

// One workgroup: the tiles blockIdx.x, blockIdx.x + gridDim.x, ... of group
// blockIdx.y, state blockIdx.z.  The stages and layouts are those of k_span; a
// term is read off the registers of the stage that holds its X mask, so a group
// of about ten masks costs one reading of the state (k_pauli: one per mask).
// partials[(b * nterms + term) * gridDim.x + blockIdx.x]
template <typename T, int LOGT, bool WIDE>
__global__ void __launch_bounds__(1 << LOGT) k_expect(const Cx<T> *__restrict__ state, uint64_t sstride,
                                                     const qs::ExpectGroup *__restrict__ groups,
                                                     const DevOp *__restrict__ all_recs,
                                                     uint32_t nterms, uint32_t ntiles, uint32_t tile_bytes,
                                                     double *__restrict__ partials) {
    using L = LdsTile<T>;
    using Off = typename OffsetOf<WIDE>::type;
    constexpr int LR = qs::kSpanRegs, E = 1 << LR, TNT = 1 << LOGT, NW = TNT / 64;
    const qs::ExpectGroup *g = groups + blockIdx.y;
    const DevOp *recs = all_recs + g->rec_begin;
    const uint32_t nrec = g->rec_end - g->rec_begin, nstage = g->stages;
    const char *st = reinterpret_cast<const char *>(state + size_t(blockIdx.z) * sstride);
    const int tid = threadIdx.x, wave = tid >> 6;
    const uint32_t ent_at = tile_bytes, lay_at = ent_at + 16u * (nrec + 1), acc_at = lay_at + kLayoutBytes * nstage;
    for (uint32_t x = uint32_t(tid); x < nrec; x += TNT) {
        const U4 *p = reinterpret_cast<const U4 *>(recs + x);
        const U4 a = p[0], c = p[1];
        U4 e = {0, 0, 0, 0};
        if (((a.w >> 16) & 0xff) == qs::DEVOP_EXPECT) {
            e.x = (a.y & 0xfu) | ((c.x & 0xfffu) << 16) | ((a.z & 0xffu) << 28);
            e.y = (c.x >> 16) | (c.y << 16);   // the sign mask of the base index
            e.z = c.y >> 16;
        } else {
            const uint32_t number = a.w >> 24;
            e.x = (kStageForm << 28) | number;
            put_layout<T>(lay_at + kLayoutBytes * number, a, c);
        }
        *reinterpret_cast<LdsU4 *>(uintptr_t(ent_at + 16u * x)) = e;
    }
    for (uint32_t x = uint32_t(tid); x < nrec * NW; x += TNT) *reinterpret_cast<LdsF8 *>(uintptr_t(acc_at + 8u * x)) = 0.0;
    __syncthreads();
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const uint64_t base = rest_base(tile, g->rest_mask);
        Cx<T> v[E];
        {
            Off off = Off(base) << L::LOGE, reg[LR];
            static_for<0, LOGT>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                off ^= ((tid >> k) & 1) ? Off(g->load_v[k]) << L::LOGE : Off(0);
            });
            static_for<0, LR>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                reg[k] = Off(g->load_v[LOGT + k]) << L::LOGE;
            });
            static_for<0, E>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                v[r] = *reinterpret_cast<const Cx<T> *>(st + (off ^ reg_off<r>(reg)));
            });
        }
        uint32_t addr[E];
        stage_addr<T, LOGT>(lay_at, tid, addr);
        if (tile != blockIdx.x && nstage > 1) __syncthreads();   // the last tile's slots have been read
        U4 ahead = lds_u4(ent_at + 16u);
        for (uint32_t i = 1; i < nrec; i++) {
            const U4 e = ahead;
            const uint32_t w = __builtin_amdgcn_readfirstlane(e.x);
            ahead = lds_u4(ent_at + 16u * (i + 1));
            const uint32_t form = w >> 28;
            if (form != kStageForm) {
                const uint32_t zl = __builtin_amdgcn_readfirstlane(e.y), zh = __builtin_amdgcn_readfirstlane(e.z);
                const uint32_t s = uint32_t(__builtin_popcount(uint32_t(tid) & ((w >> 16) & 0xfffu))) +
                                   uint32_t(__builtin_popcount(uint32_t(base) & zl)) +
                                   uint32_t(__builtin_popcount(uint32_t(base >> 32) & zh));
                const double one = flip(1.0, s << 31);
                double acc;
                switch (form) {
                case 0: acc = term_sum<T, LR, 1, false>(v, one, w); break;
                case 1: acc = term_sum<T, LR, 1, true>(v, one, w); break;
                case 2: acc = term_sum<T, LR, 2, false>(v, one, w); break;
                case 3: acc = term_sum<T, LR, 2, true>(v, one, w); break;
                case 4: acc = term_sum<T, LR, 4, false>(v, one, w); break;
                case 5: acc = term_sum<T, LR, 4, true>(v, one, w); break;
                case 6: acc = term_sum<T, LR, 8, false>(v, one, w); break;
                case 7: acc = term_sum<T, LR, 8, true>(v, one, w); break;
                default: acc = term_sum<T, LR, 0, false>(v, one, w); break;
                }
                acc = wave_total(acc);
                if ((tid & 63) == 63) *reinterpret_cast<LdsF8 *>(uintptr_t(acc_at + 8u * (i * NW + uint32_t(wave)))) += acc;
            } else {
                static_for<0, E>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    L::st(addr[r], v[r]);
                });
                stage_addr<T, LOGT>(lay_at + kLayoutBytes * (w & 0xffu), tid, addr);
                __syncthreads();
                static_for<0, E>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    v[r] = L::ld(addr[r]);
                });
            }
        }
    }
    __syncthreads();
    for (uint32_t x = uint32_t(tid); x < nrec; x += TNT) {
        if (((reinterpret_cast<const U4 *>(recs + x)[0].w >> 16) & 0xff) != qs::DEVOP_EXPECT) continue;
        double s = 0.0;
        for (int w = 0; w < NW; w++) s += *reinterpret_cast<const LdsF8 *>(uintptr_t(acc_at + 8u * (x * NW + uint32_t(w))));
        partials[(size_t(blockIdx.z) * nterms + recs[x].coef) * gridDim.x + blockIdx.x] = s;
    }
}

// ------------------------------------------------------------- launchers
namespace {
bool span_static_lds = false;

template <typename T, int LOGT, bool WIDE>
void expect_attr() {
    const void *f = reinterpret_cast<const void *>(&k_expect<T, LOGT, WIDE>);
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(max_lds_bytes()));
    if (e != hipSuccess) note_hip(e, "hipFuncSetAttribute(k_expect)");
    hipFuncAttributes fa{};
    if (hipFuncGetAttributes(&fa, f) == hipSuccess && fa.sharedSizeBytes != 0) span_static_lds = true;
}
template <typename T>
void expect_attrs() {
    expect_attr<T, 6, false>();
    expect_attr<T, 7, false>();
    expect_attr<T, 8, false>();
    expect_attr<T, 8, true>();
}

template <typename T>
int expect_t(const void *state, uint64_t sstride, uint32_t nstates, int n, const qs::ExpectPlan &plan,
             const void *table, uint32_t nterms, uint32_t chunks, uint32_t tile_bytes, size_t lds, double *partials,
             hipStream_t st) {
    const uint32_t ng = uint32_t(plan.groups.size()), ntiles = uint32_t(uint64_t(1) << (n - plan.t));
    const qs::ExpectGroup *groups = (const qs::ExpectGroup *)table;
    const DevOp *recs = reinterpret_cast<const DevOp *>(groups + ng);
    const bool wide = (uint64_t(sizeof(Cx<T>)) << n) > (uint64_t(1) << 32);
    for (uint32_t g0 = 0; g0 < ng; g0 += 32768) {   // (a grid's y extent is limited)
        const dim3 grid(chunks, std::min<uint32_t>(ng - g0, 32768), nstates);
#define QK_EXPECT(LOGT, WIDE)                                                                                   \
    hipLaunchKernelGGL((k_expect<T, LOGT, WIDE>), grid, dim3(1 << LOGT), lds, st, (const Cx<T> *)state, sstride, \
                       groups + g0, recs, nterms, ntiles, tile_bytes, partials)
        switch (plan.t - qs::kSpanRegs) {
        case 6: QK_EXPECT(6, false); break;
        case 7: QK_EXPECT(7, false); break;
        case 8:
            if (wide) QK_EXPECT(8, true);
            else QK_EXPECT(8, false);
            break;
        default: return QSIM_E_ARG;
        }
    }
#undef QK_EXPECT
    return note_hip(hipGetLastError(), "k_expect launch");
}

template <typename T, int LOGT, bool WIDE, bool MEAS, bool PAIR>
void span_attr() {
    const void *f = reinterpret_cast<const void *>(&k_span<T, LOGT, WIDE, MEAS, PAIR>);
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(max_lds_bytes()));
    if (e != hipSuccess) note_hip(e, "hipFuncSetAttribute(k_span)");
    hipFuncAttributes fa{};
    if (hipFuncGetAttributes(&fa, f) == hipSuccess && fa.sharedSizeBytes != 0) span_static_lds = true;
}
template <typename T, int LOGT>
void span_attrs() {
    span_attr<T, LOGT, false, false, false>();
    span_attr<T, LOGT, true, false, false>();
    span_attr<T, LOGT, false, true, false>();
    span_attr<T, LOGT, false, false, true>();
    span_attr<T, LOGT, true, false, true>();
    span_attr<T, LOGT, false, true, true>();
}

struct SpanLaunch {
    void *state;
    uint64_t sstride;
    uint32_t nstates;
    const SpanArgs &sa;
    const DevOp *ops;
    uint32_t ob, oe;
    const void *coefs;
    uint32_t cb;
    uint64_t cstride;
    const MeasArgs &ma;
    uint32_t flags;
    size_t lds;
    hipStream_t st;

    template <typename T, int LOGT, bool WIDE, bool MEAS>
    void kernel() const {
        const dim3 grid(uint32_t(uint64_t(1) << (sa.n - sa.t)), nstates);
        if (sa.pairs)
            hipLaunchKernelGGL((k_span<T, LOGT, WIDE, MEAS, true>), grid, dim3(1 << LOGT), lds, st, (Cx<T> *)state,
                               sstride, sa, ops, ob, oe, (const Cx<T> *)coefs, cb, cstride, ma, flags);
        else
            hipLaunchKernelGGL((k_span<T, LOGT, WIDE, MEAS, false>), grid, dim3(1 << LOGT), lds, st, (Cx<T> *)state,
                               sstride, sa, ops, ob, oe, (const Cx<T> *)coefs, cb, cstride, ma, flags);
    }
    template <typename T, int LOGT>
    void tile() const {
        // (a whole state in one tile, the place of measurement records, is narrow)
        if ((uint64_t(sizeof(Cx<T>)) << sa.n) > (uint64_t(1) << 32)) kernel<T, LOGT, true, false>();
        else if (sa.nrun < oe - ob) kernel<T, LOGT, false, true>();
        else kernel<T, LOGT, false, false>();
    }
    template <typename T>
    int run() const {
        switch (sa.t - qs::kSpanRegs) {
        case 6: tile<T, 6>(); break;
        case 7: tile<T, 7>(); break;
        case 8: tile<T, 8>(); break;
        case 9: tile<T, 9>(); break;
        case 10:
            // (a complex128 tile of 14 dimensions is larger than the LDS)
            if constexpr (sizeof(T) == 4) {
                tile<T, 10>();
                break;
            }
            return QSIM_E_CAPACITY;
        default: return QSIM_E_ARG;
        }
        return note_hip(hipGetLastError(), "k_span launch");
    }
};
}  // namespace

bool init_span_kernels() {
    span_attrs<float, 6>();
    span_attrs<float, 7>();
    span_attrs<float, 8>();
    span_attrs<float, 9>();
    span_attrs<float, 10>();
    span_attrs<double, 6>();
    span_attrs<double, 7>();
    span_attrs<double, 8>();
    span_attrs<double, 9>();
    expect_attrs<float>();
    expect_attrs<double>();
    (void)hipGetLastError();
    return !span_static_lds;
}

// Workgroups per group and state: up to 1024, fewer for many terms and states,
// so that the partial sums stay within 32 MiB.
uint32_t expect_chunks(int n, int t, uint32_t nterms, uint32_t nstates) {
    uint64_t c = std::min<uint64_t>(uint64_t(1) << (n - t), 1024);
    while (c > 1 && c * nterms * nstates > (uint64_t(1) << 22)) c /= 2;
    return uint32_t(c);
}

int launch_expect(int dtype, const void *state, uint64_t sstride, uint32_t nstates, int n, const qs::ExpectPlan &plan,
                  const void *table, uint32_t nterms, uint32_t chunks, double *partials, double *out,
                  hipStream_t st) {
    const size_t elem = dtype == QSIM_C64 ? 8 : 16;
    if (!qs::span_tile_ok(plan.t) || plan.t > 12 || plan.t > n || n - plan.t > 31 || plan.groups.empty() ||
        chunks == 0 || chunks > (uint64_t(1) << (n - plan.t)))
        return QSIM_E_ARG;
    const uint32_t tile_bytes = plan.relaid ? uint32_t(elem << plan.t) : 0u;
    const size_t nw = (size_t(1) << (plan.t - qs::kSpanRegs)) / 64;
    const size_t lds = tile_bytes + 16 * (size_t(plan.max_rec) + 1) + kLayoutBytes * size_t(plan.max_stage) + 8 * nw * plan.max_rec;
    if (lds > max_lds_bytes()) return QSIM_E_CAPACITY;
    const int rc = dtype == QSIM_C64 ? expect_t<float>(state, sstride, nstates, n, plan, table, nterms, chunks,
                                                       tile_bytes, lds, partials, st)
                                     : expect_t<double>(state, sstride, nstates, n, plan, table, nterms, chunks,
                                                        tile_bytes, lds, partials, st);
    if (rc) return rc;
    launch_finish(partials, chunks, nstates * nterms, out, st);
    return note_hip(hipGetLastError(), "k_finish launch");
}

int launch_span(int dtype, void *state, uint64_t sstride, uint32_t nstates, const SpanArgs &sa, const DevOp *ops,
                uint32_t ob, uint32_t oe, const void *coefs, uint32_t cb, uint64_t cstride, const MeasArgs &ma,
                uint32_t flags, hipStream_t st) {
    const size_t elem = dtype == QSIM_C64 ? 8 : 16;
    if (!qs::span_tile_ok(sa.t) || sa.t > sa.n || sa.n - sa.t > 31 || oe <= ob || sa.nlayout == 0 ||
        sa.nlayout > oe - ob || sa.nrun == 0 || sa.nrun > oe - ob || (sa.nrun < oe - ob && sa.t != sa.n) ||
        (sa.tile_bytes != 0 && sa.tile_bytes != (elem << sa.t)))
        return QSIM_E_ARG;
    // records write the states' status, and their outcomes where there are slots
    if (sa.nrun < oe - ob && (!ma.status || (ma.nslots > 0 && (!ma.outcomes || !ma.probs)))) return QSIM_E_ARG;
    const size_t lds = span_lds_bytes(sa.tile_bytes, oe - ob, sa.nlayout);
    if (lds > max_lds_bytes()) return QSIM_E_CAPACITY;
    const SpanLaunch l{state, sstride, nstates, sa, ops, ob, oe, coefs, cb, cstride, ma, flags, lds, st};
    return dtype == QSIM_C64 ? l.run<float>() : l.run<double>();
}

}  // namespace qk
