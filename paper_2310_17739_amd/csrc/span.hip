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
// Plain loads and stores: non-temporal ones, which suit k_tile's passes, cost
// 1540 us against 925 per pass at 27 qubits complex128 and 5174 against 3681 at
// 30 qubits complex64 (22.1 against 19.4 at 21 qubits complex128).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"
#include "launch.h"

namespace qk {

using qs::DevOp;

// v with its sign flipped where bit 31 of s is set
__device__ __forceinline__ float flip(float v, uint32_t s) { return __uint_as_float(__float_as_uint(v) ^ s); }
__device__ __forceinline__ double flip(double v, uint32_t s) {
    return __longlong_as_double(__double_as_longlong(v) ^ (int64_t(uint64_t(s) << 32)));
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

// The sign bit that turns pair k's t into pair k + 1's: bit k + 1 of d.
__device__ __forceinline__ uint32_t turn_sign(uint32_t d, int k) { return (d << (31 - k)) & 0x80000000u; }

// One rotation from a thread's registers x to y, y[r] = x[r] + t_r x[r ^ M] with
// M one register bit or none, t real (REAL) or imaginary.  t has the sign of
// register 0 (and of the tile and the thread); the pairs {r, r ^ M} follow in
// ascending order of their smaller register, and bit k of d tells whether pair
// k's sign differs from that of pair k - 1, so that a sign costs one operation
// on one register.  Register r ^ M has the sign of r for an imaginary t (an
// even number of Y letters) and the opposite one for a real t.
template <typename T, int LR, int M, bool REAL>
__device__ __forceinline__ void rotate(const Cx<T> (&x)[1 << LR], Cx<T> (&y)[1 << LR], T t, uint32_t d) {
    static_for<0, 1 << LR>([&](auto rc) {
        constexpr int r = decltype(rc)::value, q = r ^ M;
        if constexpr (M == 0 || r < q) {
            // place of the pair in the order
            constexpr int k = M == 0 ? r : (r / (2 * M)) * M + r % M;
            if constexpr (k > 0) t = flip(t, turn_sign(d, k));
            const Cx<T> a = x[r], b = x[q];
            if constexpr (REAL) {
                y[r] = Cx<T>{T(fma(t, b.re, a.re)), T(fma(t, b.im, a.im))};
                y[q] = Cx<T>{T(fma(-t, a.re, b.re)), T(fma(-t, a.im, b.im))};
            } else {
                y[r] = Cx<T>{T(fma(-t, b.im, a.re)), T(fma(t, b.re, a.im))};
                if constexpr (M != 0) y[q] = Cx<T>{T(fma(-t, a.im, b.re)), T(fma(t, a.re, b.im))};
            }
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

// LDS byte addresses of a layout (a stage record): the thread's part and
// each register bit's.
template <typename T, int LOGT>
__device__ __forceinline__ void stage_layout(const uint32_t (&w)[8], int tid, uint32_t &slot_t,
                                             uint32_t (&slot_r)[qs::kSpanRegs]) {
    constexpr int LOGE = LdsTile<T>::LOGE;
    const uint32_t h[14] = {w[0] & 0xffff, w[0] >> 16,    w[1] & 0xffff, w[1] >> 16,    w[2] & 0xffff,
                            w[2] >> 16,    w[3] & 0xffff, w[4] & 0xffff, w[4] >> 16,    w[5] & 0xffff,
                            w[5] >> 16,    w[6] & 0xffff, w[6] >> 16,    w[7] & 0xffff};
    slot_t = 0;
    static_for<0, LOGT>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        slot_t ^= ((tid >> k) & 1) ? h[k] << LOGE : 0;
    });
    static_for<0, qs::kSpanRegs>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        slot_r[k] = h[LOGT + k] << LOGE;
    });
}

template <typename T, int LOGT>
__global__ void __launch_bounds__(1 << LOGT) k_span(Cx<T> *__restrict__ state, uint64_t sstride, SpanArgs sa,
                                                   const DevOp *__restrict__ ops, uint32_t ob, uint32_t oe,
                                                   const Cx<T> *__restrict__ coefs, uint32_t cb, uint32_t ce,
                                                   uint64_t cstride, const int32_t *__restrict__ status,
                                                   uint32_t flags) {
    using L = LdsTile<T>;
    constexpr int LR = qs::kSpanRegs, E = 1 << LR, TNT = 1 << LOGT;
    const uint32_t b = blockIdx.y;
    if (status && status[b] != 0) return;   // an earlier step of this state failed
    Cx<T> *st = state + size_t(b) * sstride;
    const Cx<T> *gcf = coefs + size_t(b) * cstride + cb;
    const int tid = threadIdx.x;
    const uint32_t nrec = oe - ob, ncf = ce - cb;
    // LDS: the tile (unless the pass has a single stage), records, coefficients
    const uint32_t rec_at = sa.tile_bytes, cf_at = rec_at + nrec * uint32_t(sizeof(DevOp));
    const uint64_t base = span_base(blockIdx.x, sa);
    typedef uint32_t U4 __attribute__((ext_vector_type(4)));

    Cx<T> v[E];
    {
        uint64_t off = base;
#pragma unroll
        for (int k = 0; k < LOGT; k++) off ^= ((tid >> k) & 1) ? sa.load_v[k] : 0;
        if (flags & TF_INIT_ZERO) {
            static_for<0, E>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                v[r] = Cx<T>{T((off ^ reg_off<r>(sa.load_v + LOGT)) == 0 ? 1 : 0), T(0)};
            });
        } else {
            static_for<0, E>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                v[r] = st[off ^ reg_off<r>(sa.load_v + LOGT)];
            });
        }
    }
    // the pass's records and coefficients follow while the tile loads fly
    const U4 *gops = reinterpret_cast<const U4 *>(ops + ob);
    for (uint32_t x = uint32_t(tid); x < 2 * nrec; x += TNT)
        *reinterpret_cast<__attribute__((address_space(3))) U4 *>(uintptr_t(rec_at + 16u * x)) = gops[x];
    for (uint32_t x = uint32_t(tid); x < ncf; x += TNT) L::st(cf_at + (x << L::LOGE), gcf[x]);
    __syncthreads();

    double scale = 1.0;
    uint32_t slot_t = 0, slot_r[LR] = {};   // LDS bytes: the thread's part, each register bit's
    auto rec = [&](uint32_t i, U4 &a, U4 &c) {
        a = *reinterpret_cast<const __attribute__((address_space(3))) U4 *>(uintptr_t(rec_at + 32u * i));
        c = *reinterpret_cast<const __attribute__((address_space(3))) U4 *>(uintptr_t(rec_at + 32u * i + 16u));
    };
    U4 ra, rb;
    rec(0, ra, rb);
    uint32_t cf = cf_at;
    Cx<T> e0 = L::ld(cf), e1 = L::ld(cf + uint32_t(sizeof(Cx<T>)));
    // One record, from the registers x to y.  (Two sets of registers in turn:
    // a rotation reads both members of a pair for both results, and in one set
    // every second result would have to be moved.)
    auto step = [&](uint32_t i, const Cx<T> (&x)[E], Cx<T> (&y)[E]) __attribute__((always_inline)) {
        uint32_t w[8] = {ra.x, ra.y, ra.z, ra.w, rb.x, rb.y, rb.z, rb.w};
#pragma unroll
        for (int j = 0; j < 8; j++) w[j] = __builtin_amdgcn_readfirstlane(w[j]);
        const bool pauli = ((w[3] >> 16) & 0xff) == qs::DEVOP_PAULI;
        const Cx<T> c0 = e0, c1 = e1;
        // the next record and (rotations take theirs in order) coefficients;
        // what the last one reads lies inside the padding of the LDS block
        if (pauli) cf += 2u * uint32_t(sizeof(Cx<T>));
        rec(i + 1, ra, rb);
        e0 = L::ld(cf);
        e1 = L::ld(cf + uint32_t(sizeof(Cx<T>)));
        if (pauli) {
            const uint64_t zb = uint64_t((w[4] >> 16) | (w[5] << 16)) | (uint64_t(w[5] >> 16) << 32);
            const uint32_t s = uint32_t(__builtin_popcount(uint32_t(tid) & (w[4] & 0xffffu))) +
                               uint32_t(__builtin_popcountll(base & zb));
            scale *= double(c0.re) + double(c0.im);
            rotate_form<T, LR>(x, y, int(w[2] & 0xff), flip(c1.im, s << 31), w[1]);
            // a factor that the pass's scale does not take (the same on every lane)
            if (__builtin_amdgcn_readfirstlane(int(c1.re != T(0)))) {
                static_for<0, E>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    y[r].re *= c1.re;
                    y[r].im *= c1.re;
                });
            }
        } else {
            // a stage: through LDS into its layout
            static_for<0, E>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                L::st(slot_t ^ reg_off<r>(slot_r), x[r]);
            });
            stage_layout<T, LOGT>(w, tid, slot_t, slot_r);
            __syncthreads();
            static_for<0, E>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                y[r] = L::ld(slot_t ^ reg_off<r>(slot_r));
            });
        }
    };
    {
        // the first record: the layout of the load
        uint32_t w[8] = {ra.x, ra.y, ra.z, ra.w, rb.x, rb.y, rb.z, rb.w};
#pragma unroll
        for (int j = 0; j < 8; j++) w[j] = __builtin_amdgcn_readfirstlane(w[j]);
        stage_layout<T, LOGT>(w, tid, slot_t, slot_r);
        rec(1, ra, rb);
    }
    uint32_t i = 1;
    for (; i + 1 < nrec; i += 2) {
        Cx<T> u[E];
        step(i, v, u);
        step(i + 1, u, v);
    }
    if (i < nrec) {
        Cx<T> u[E];
        step(i, v, u);
        static_for<0, E>([&](auto rc) { v[decltype(rc)::value] = u[decltype(rc)::value]; });
    }
    {
        uint64_t off = base;
#pragma unroll
        for (int k = 0; k < LOGT; k++) off ^= ((tid >> k) & 1) ? sa.store_v[k] : 0;
        const T fr = T(scale * sa.phase_re), fi = T(scale * sa.phase_im);
        const bool turned = sa.phase_im != 0.0;
        static_for<0, E>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            Cx<T> y{v[r].re * fr, v[r].im * fr};
            if (turned) {
                y.re = fma(-fi, v[r].im, y.re);
                y.im = fma(fi, v[r].re, y.im);
            }
            st[off ^ reg_off<r>(sa.store_v + LOGT)] = y;
        });
    }
}

// ------------------------------------------------------------- launchers
namespace {
bool span_static_lds = false;

template <typename T, int LOGT>
void span_attr() {
    const void *f = reinterpret_cast<const void *>(&k_span<T, LOGT>);
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(max_lds_bytes()));
    if (e != hipSuccess) note_hip(e, "hipFuncSetAttribute(k_span)");
    hipFuncAttributes fa{};
    if (hipFuncGetAttributes(&fa, f) == hipSuccess && fa.sharedSizeBytes != 0) span_static_lds = true;
}

template <typename T>
int span_t(void *state, uint64_t sstride, uint32_t nstates, const SpanArgs &sa, const DevOp *ops, uint32_t ob,
           uint32_t oe, const void *coefs, uint32_t cb, uint32_t ce, uint64_t cstride, const int32_t *status,
           uint32_t flags, size_t lds, hipStream_t st) {
    const dim3 grid(uint32_t(uint64_t(1) << (sa.n - sa.t)), nstates);
#define QK_SPAN(LOGT)                                                                                          \
    case LOGT:                                                                                                 \
        hipLaunchKernelGGL((k_span<T, LOGT>), grid, dim3(1 << LOGT), lds, st, (Cx<T> *)state, sstride, sa, ops, \
                           ob, oe, (const Cx<T> *)coefs, cb, ce, cstride, status, flags);                      \
        break;
    switch (sa.t - qs::kSpanRegs) {
        QK_SPAN(6)
        QK_SPAN(7)
        QK_SPAN(8)
        QK_SPAN(9)
    case 10:
        // (a complex128 tile of 14 dimensions is larger than the LDS)
        if constexpr (sizeof(T) == 4) {
            hipLaunchKernelGGL((k_span<T, 10>), grid, dim3(1 << 10), lds, st, (Cx<T> *)state, sstride, sa, ops, ob,
                               oe, (const Cx<T> *)coefs, cb, ce, cstride, status, flags);
            break;
        }
        return QSIM_E_CAPACITY;
    default: return QSIM_E_ARG;
    }
#undef QK_SPAN
    return note_hip(hipGetLastError(), "k_span launch");
}
}  // namespace

bool init_span_kernels() {
    span_attr<float, 6>();
    span_attr<float, 7>();
    span_attr<float, 8>();
    span_attr<float, 9>();
    span_attr<float, 10>();
    span_attr<double, 6>();
    span_attr<double, 7>();
    span_attr<double, 8>();
    span_attr<double, 9>();
    (void)hipGetLastError();
    return !span_static_lds;
}

int launch_span(int dtype, void *state, uint64_t sstride, uint32_t nstates, const SpanArgs &sa, const DevOp *ops,
                uint32_t ob, uint32_t oe, const void *coefs, uint32_t cb, uint32_t ce, uint64_t cstride,
                const int32_t *status, uint32_t flags, hipStream_t st) {
    const size_t elem = dtype == QSIM_C64 ? 8 : 16;
    if (!qs::span_tile_ok(sa.t) || sa.t > sa.n || sa.n - sa.t > 31 || oe <= ob || ce < cb ||
        (sa.tile_bytes != 0 && sa.tile_bytes != (elem << sa.t)))
        return QSIM_E_ARG;
    const size_t lds = span_lds_bytes(elem, sa.tile_bytes, oe - ob, ce - cb);
    if (lds > max_lds_bytes()) return QSIM_E_CAPACITY;
    return dtype == QSIM_C64 ? span_t<float>(state, sstride, nstates, sa, ops, ob, oe, coefs, cb, ce, cstride, status,
                                             flags, lds, st)
                             : span_t<double>(state, sstride, nstates, sa, ops, ob, oe, coefs, cb, ce, cstride, status,
                                              flags, lds, st);
}

}  // namespace qk
