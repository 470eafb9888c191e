// Host emulation of compiled plans (qsim_debug_emulate*): what the kernels do with
// a plan's device tables, in FP64 on the host, for tests without a GPU.
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "host.h"
#include "launch.h"
#include "runtime.h"

using namespace qs;

namespace {

// Measurement records of one state: inputs, outputs and the first failure.
struct Records {
    const double *uniforms = nullptr;
    const int32_t *forced = nullptr;
    int32_t *outcomes = nullptr;
    double *probs = nullptr;
    int status = QSIM_OK;

    // The decision on weights P0, P1: *o is the value kept, *scale what its
    // amplitudes are multiplied by, *move whether the values change places then.
    // Returns QSIM_OK or the failure, which is also the state's status.
    int decide(int kind, int slot, double P0, double P1, int *o, double *scale, bool *move) {
        *scale = 1.0;
        *move = false;
        *o = -1;
        if (kind == DEVOP_RESET) {
            if (P1 == 0.0) return QSIM_OK;
            if (P0 != 0.0) return status = QSIM_E_NOT_DEFINITE;
            *move = true;
            return QSIM_OK;
        }
        if (kind == DEVOP_ASSERT0) {
            if (!(P0 > 0.0)) return status = QSIM_E_ZERO_PROB;
            *o = 0;
        } else if (forced && forced[slot] >= 0) {
            *o = forced[slot];
            if (!((*o ? P1 : P0) > 0.0)) return status = QSIM_E_ZERO_PROB;
        } else {
            *o = uniforms[slot] < P0 / (P0 + P1) ? 0 : 1;
        }
        const double kept = *o ? P1 : P0;
        if (outcomes) outcomes[slot] = *o;
        if (probs) probs[slot] = kept / (P0 + P1);
        *scale = 1.0 / std::sqrt(kept);
        *move = kind == DEVOP_MEASURE_RESET && *o;
        return QSIM_OK;
    }

    // A record of an array whose entry i has the value value(i), changed by flip(i).
    template <typename V, typename F>
    int run(int kind, int slot, std::size_t len, cd *v, V &&value, F &&flip) {
        double P[2] = {0.0, 0.0};
        for (std::size_t i = 0; i < len; i++) P[value(i)] += std::norm(v[i]);
        int o;
        double f;
        bool move;
        const int rc = decide(kind, slot, P[0], P[1], &o, &f, &move);
        if (rc) return rc;
        if (o >= 0)
            for (std::size_t i = 0; i < len; i++) v[i] = int(value(i)) == o ? v[i] * f : cd(0.0);
        if (move)
            for (std::size_t i = 0; i < len; i++)
                if (!value(i)) std::swap(v[i], v[flip(i)]);
        return QSIM_OK;
    }
};

// The passes of c on the state st (2^n amplitudes); `recs`: as a batch runs them,
// with measurement records, up to the first that fails.
int emulate(int n, const Compiled &c, cd *st, Records *recs) {
    const PackedPlan &p = c.plan;
    // y[r] = sum over present shifts (ascending) of cf[term * 2^k + r] x[r ^ m]
    // on the 2^k members of every group of a width-w array addressed by pos[]
    auto apply = [&](cd *v, int w, const DevOp &o, const cd *cf) {
        const int k = o.k, d = 1 << k;
        std::vector<cd> x(d), y(d);
        for (uint64_t grp = 0; grp < (uint64_t(1) << (w - k)); grp++) {
            uint64_t b0 = grp;
            for (int j = 0; j < k; j++)
                b0 = ((b0 >> o.pos[j]) << (o.pos[j] + 1)) | (b0 & ((uint64_t(1) << o.pos[j]) - 1));
            auto at = [&](int r) {
                uint64_t a = b0;
                for (int j = 0; j < k; j++)
                    if ((r >> j) & 1) a |= uint64_t(1) << o.pos[j];
                return a;
            };
            for (int r = 0; r < d; r++) x[r] = v[at(r)];
            for (int r = 0; r < d; r++) {
                cd acc = 0;
                int term = 0;
                for (int m = 0; m < d; m++)
                    if ((o.present >> m) & 1) acc += cf[size_t(term++) * d + r] * x[r ^ m];
                y[r] = acc;
            }
            for (int r = 0; r < d; r++) v[at(r)] = y[r];
        }
    };
    for (size_t i = 0; i < c.passes.size(); i++) {
        const PassInfo &pi = c.passes[i];
        if (recs && recs->status) break;   // the state's later passes return at once
        if (pi.kind == Pass::MEASURE) {
            if (!recs) return QSIM_E_ARG;
            const uint64_t bit = uint64_t(1) << pi.meas.q;
            recs->run(pi.meas.kind, pi.meas.slot, size_t(1) << n, st, [&](uint64_t x) { return (x & bit) != 0; },
                      [&](uint64_t x) { return x ^ bit; });
            continue;
        }
        if (pi.strided) {
            for (uint32_t j = p.pass_begin[i]; j < p.pass_begin[i + 1]; j++) {
                const DevOp &o = p.ops[j];
                if (o.kind != DEVOP_MAT || o.kx) return QSIM_E_ARG;
                apply(st, n, o, p.coefs.data() + o.coef);
            }
            continue;
        }
        if (pi.reg) {
            // register-resident pass: elements indexed by position bits
            // (thread bits, then register bits), moved as the kernel moves them
            const qk::RegArgs &ra = pi.ra;
            const int t = ra.t, logt = t - kRegBits;
            std::vector<cd> v(size_t(1) << t), w(v.size());
            for (uint64_t tile = 0; tile < (uint64_t(1) << (n - t)); tile++) {
                const uint64_t base = qk::tile_base(tile, ra.rest_mask, ra.nxcd, ra.xcd_q);
                auto addr = [&](uint64_t P, const uint8_t *pos) {
                    uint64_t a = base;
                    for (int b = 0; b < t; b++)
                        if ((P >> b) & 1) a |= uint64_t(1) << ra.tq[pos[b]];
                    return a;
                };
                uint8_t cur[16];
                std::memcpy(cur, ra.load_pos, 16);
                for (uint64_t P = 0; P < v.size(); P++) v[P] = st[addr(P, ra.load_pos)];
                for (uint32_t j = p.pass_begin[i]; j < p.pass_begin[i + 1]; j++) {
                    const DevOp &o = p.ops[j];
                    if (o.kind == DEVOP_RMAT) {
                        uint32_t e = 0;
                        for (int x = 0; x < o.kx; x++) e |= uint32_t((base >> o.xq[x]) & 1) << x;
                        const cd *cf = p.coefs.data() + o.coef + (size_t(e) * __builtin_popcount(o.present) << 4);
                        for (uint64_t tid = 0; tid < (uint64_t(1) << logt); tid++) {
                            cd x[16], y[16];
                            for (int r = 0; r < 16; r++) x[r] = v[tid | (uint64_t(r) << logt)];
                            for (int r = 0; r < 16; r++) {
                                cd acc = 0;
                                int term = 0;
                                for (int M = 0; M < 16; M++)
                                    if ((o.present >> M) & 1) acc += cf[size_t(term++) * 16 + r] * x[r ^ M];
                                y[r] = acc;
                            }
                            for (int r = 0; r < 16; r++) v[tid | (uint64_t(r) << logt)] = y[r];
                        }
                    } else if (o.kind == DEVOP_SWAP) {
                        const int a = o.pos[0], b = logt + o.pos[1];
                        for (uint64_t P = 0; P < v.size(); P++) {
                            const uint64_t ba = (P >> a) & 1, bb = (P >> b) & 1;
                            uint64_t Q = P & ~((uint64_t(1) << a) | (uint64_t(1) << b));
                            Q |= (ba << b) | (bb << a);
                            w[Q] = v[P];
                        }
                        std::swap(v, w);
                        std::swap(cur[a], cur[b]);
                    } else if (o.kind == DEVOP_XPOSE && j + 1 < p.pass_begin[i + 1]) {
                        const uint8_t *from = reinterpret_cast<const uint8_t *>(&o);
                        const uint8_t *to = reinterpret_cast<const uint8_t *>(&p.ops[j + 1]);
                        if (std::memcmp(from, cur, size_t(t)) != 0) return QSIM_E_ARG;
                        int to_pos[16];
                        for (int b = 0; b < t; b++) to_pos[to[b]] = b;
                        for (uint64_t P = 0; P < v.size(); P++) {
                            uint64_t Q = 0;
                            for (int b = 0; b < t; b++)
                                if ((P >> b) & 1) Q |= uint64_t(1) << to_pos[from[b]];
                            w[Q] = v[P];
                        }
                        std::swap(v, w);
                        std::memcpy(cur, to, size_t(t));
                        j++;
                    } else {
                        return QSIM_E_ARG;
                    }
                }
                if (std::memcmp(cur, ra.store_pos, size_t(t)) != 0) return QSIM_E_ARG;
                for (uint64_t P = 0; P < v.size(); P++) st[addr(P, ra.store_pos)] = v[P];
            }
            continue;
        }
        if (pi.span) {
            // elements at positions (thread bits, then register bits), moved
            // through the slots of each stage's layout
            const qk::SpanArgs &sa = pi.sa;
            const int t = sa.t, logt = t - kSpanRegs;
            auto combine = [&](uint64_t P, auto &&vec) {
                uint64_t a = 0;
                for (int b = 0; b < t; b++)
                    if ((P >> b) & 1) a ^= uint64_t(vec(b));
                return a;
            };
            // the words of a stage's or a layout's record
            auto slots = [](const uint8_t *at) {
                return [at](int x) {
                    uint16_t s;
                    std::memcpy(&s, at + (x < 7 ? 2 * x : 16 + 2 * (x - 7)), 2);
                    return s;
                };
            };
            std::vector<cd> v(size_t(1) << t), w(v.size());
            const cd turn(sa.phase_re, sa.phase_im);
            for (uint64_t tile = 0; tile < (uint64_t(1) << (n - t)); tile++) {
                const uint64_t base = qk::span_base(tile, sa);
                for (uint64_t P = 0; P < v.size(); P++) v[P] = st[base ^ combine(P, [&](int b) { return sa.load_v[b]; })];
                const uint8_t *cur = nullptr, *failed = nullptr;
                cd scale = 1.0;
                for (uint32_t j = p.pass_begin[i]; j < p.pass_begin[i] + sa.nrun; j++) {
                    const DevOp &o = p.ops[j];
                    if (o.kind == DEVOP_SPAN_REC) {
                        if (!recs) return QSIM_E_ARG;
                        const uint32_t dir = (o.present >> 4) & 7;
                        auto value = [&](uint64_t P) {
                            return ((__builtin_popcountll(P & ((uint64_t(1) << logt) - 1) & o.slot[0]) +
                                     __builtin_popcountll((P >> logt) & (o.present & 15)) + int((o.present >> 7) & 1)) & 1) != 0;
                        };
                        if (!recs->run(o.pos[0], int(o.slot[1] | uint32_t(o.slot[2]) << 16), v.size(), v.data(), value,
                                       [&](uint64_t P) { return dir ? P ^ (uint64_t(1) << (logt + dir - 1)) : P; })) {
                            // a collapse leaves norm 1; what the scale holds is its sign
                            if (o.pos[0] != DEVOP_RESET) scale = scale.real() < 0.0 ? -1.0 : 1.0;
                            continue;
                        }
                        for (uint32_t l = p.pass_begin[i] + sa.nrun; l < p.pass_begin[i + 1]; l++)
                            if (p.ops[l].kx == o.kx) failed = reinterpret_cast<const uint8_t *>(&p.ops[l]);
                        if (!failed) return QSIM_E_ARG;
                        break;
                    }
                    if (o.kind == DEVOP_STAGE) {
                        const uint8_t *raw = reinterpret_cast<const uint8_t *>(&o);
                        if (cur) {
                            for (uint64_t P = 0; P < v.size(); P++) w[combine(P, slots(cur))] = v[P];
                            for (uint64_t P = 0; P < v.size(); P++) v[P] = w[combine(P, slots(raw))];
                        }
                        cur = raw;
                        continue;
                    }
                    const uint64_t zb = uint64_t(o.slot[1]) | uint64_t(o.slot[2]) << 16 | uint64_t(o.slot[3]) << 32;
                    auto parity = [&](uint64_t P, const DevOp &m, uint64_t mb) {
                        const uint64_t tid = P & ((uint64_t(1) << logt) - 1), r = P >> logt;
                        return (__builtin_popcountll(tid & m.slot[0]) + __builtin_popcountll(base & mb) +
                                __builtin_popcountll(r & m.present)) & 1;
                    };
                    const cd e0 = p.coefs[o.coef], e1 = p.coefs[o.coef + 1];
                    if (o.kind == DEVOP_PAULI2) {
                        const DevOp &m = p.ops[j + 1];
                        const uint64_t wb = uint64_t(m.slot[1]) | uint64_t(m.slot[2]) << 16 | uint64_t(m.slot[3]) << 32;
                        for (uint64_t P = 0; P < v.size(); P++) {
                            const cd c = parity(P, m, wb) ? e1 : e0;
                            const double A = c.real(), B = parity(P, o, zb) ? -c.imag() : c.imag();
                            const cd a = v[P], b = v[P ^ (uint64_t(1) << (logt + (o.k >> 1)))];
                            w[P] = (o.k & 1) ? cd(std::fma(B, b.real(), A * a.real()), std::fma(B, b.imag(), A * a.imag()))
                                             : cd(std::fma(-B, b.imag(), A * a.real()), std::fma(B, b.real(), A * a.imag()));
                        }
                        std::swap(v, w);
                        j += 2;
                        continue;
                    }
                    scale *= e0.real() + e0.imag();
                    const bool diag = o.k == 2 * kSpanRegs, real = !diag && (o.k & 1);
                    const uint32_t m = diag ? 0u : 1u << (o.k >> 1);
                    for (uint64_t P = 0; P < v.size(); P++) {
                        const double tt = parity(P, o, zb) ? -e1.imag() : e1.imag();
                        const cd a = v[P], b = v[P ^ (uint64_t(m) << logt)];
                        w[P] = real ? cd(std::fma(tt, b.real(), a.real()), std::fma(tt, b.imag(), a.imag()))
                                    : cd(std::fma(-tt, b.imag(), a.real()), std::fma(tt, b.real(), a.imag()));
                        if (e1.real() != 0.0) w[P] *= scale;
                    }
                    if (e1.real() != 0.0) scale = 1.0;
                    std::swap(v, w);
                }
                scale *= turn;
                if (failed) {
                    for (uint64_t P = 0; P < v.size(); P++) st[combine(P, slots(failed)) ^ slots(failed)(14)] = v[P] * scale;
                    continue;
                }
                for (uint64_t P = 0; P < v.size(); P++)
                    st[base ^ sa.store_base ^ combine(P, [&](int b) { return sa.store_v[b]; })] = v[P] * scale;
            }
            continue;
        }
        const qk::TileArgs &ta = pi.ta;
        const int t = ta.t;
        std::vector<cd> v(size_t(1) << t);
        for (uint64_t tile = 0; tile < (uint64_t(1) << (n - t)); tile++) {
            // the workgroup's tile in the kernel's order
            const uint64_t base = qk::tile_base(tile, ta.rest_mask, ta.nxcd, ta.xcd_q);
            auto addr = [&](uint64_t jpos) {
                uint64_t a = base;
                for (int b = 0; b < t; b++)
                    if ((jpos >> b) & 1) a |= uint64_t(1) << ta.tq[b];
                return a;
            };
            for (uint64_t jpos = 0; jpos < v.size(); jpos++) v[jpos] = st[addr(jpos)];
            for (uint32_t j = p.pass_begin[i]; j < p.pass_begin[i + 1]; j++) {
                const DevOp &o = p.ops[j];
                if (o.kind == DEVOP_RUN) continue;   // its operators follow
                if (recs && devop_is_record(o.kind)) {
                    const uint64_t bit = uint64_t(1) << o.pos[0];
                    if (recs->run(o.kind, int(o.coef), v.size(), v.data(), [&](uint64_t x) { return (x & bit) != 0; },
                                  [&](uint64_t x) { return x ^ bit; }))
                        break;
                    continue;
                }
                if (o.kind != DEVOP_MAT) return QSIM_E_ARG;
                uint32_t e = 0;
                for (int x = 0; x < o.kx; x++) e |= uint32_t((base >> o.xq[x]) & 1) << x;
                apply(v.data(), t, o,
                      p.coefs.data() + o.coef + size_t(e) * (size_t(__builtin_popcount(o.present)) << o.k));
            }
            for (uint64_t jpos = 0; jpos < v.size(); jpos++) st[addr(jpos)] = v[jpos];
        }
    }
    return QSIM_OK;
}

// Coefficients of one state of a template, as k_bind computes them.
void bind_coefs(Compiled *c, const std::vector<qk::BindEntry> &ents, const double *params, bool single, size_t ncoef) {
    std::vector<cd> out(ncoef);
    const std::vector<cd> &tmpl = c->plan.coefs;
    for (const qk::BindEntry &e : ents) {
        if (e.np < 0) {
            const double th = params[e.slot[0]];
            const double s = tmpl[e.tmpl_off].real() * std::sin(0.5 * th);
            cd y[2];
            pauli_coefs(std::cos(0.5 * th), s, single, y);
            if (!(std::fabs(s) <= std::fabs(std::cos(0.5 * th)))) y[1] = cd(1.0, y[1].imag());
            out[e.bound_off] = y[0];
            out[e.bound_off + 1] = y[1];
            continue;
        }
        for (uint32_t i = 0; i < e.count; i++) {
            cd acc = 0.0;
            for (int sb = 0; sb < (1 << e.np); sb++) {
                double w = 1.0;
                for (int j = 0; j < e.np; j++)
                    w *= ((sb >> j) & 1) ? std::sin(0.5 * params[e.slot[j]]) : std::cos(0.5 * params[e.slot[j]]);
                acc += w * tmpl[size_t(e.tmpl_off) + size_t(sb) * e.count + i];
            }
            out[e.bound_off + i] = acc;
        }
    }
    c->plan.coefs.swap(out);
}

}  // namespace

extern "C" {

int qsim_debug_emulate(int n, int dtype, const qsim_gate *g, size_t ng, const double *mats,
                       size_t n_mats, const double *params, size_t n_params,
                       const qsim_fuse_opts *opt, double *psi) {
    if (n < 1 || n > 24 || (dtype != QSIM_C64 && dtype != QSIM_C128) || (ng && !g) || !psi) return QSIM_E_ARG;
    try {
        Compiled c;
        const int rc = compile_circuit(n, dtype, g, ng, GateInputs{mats, n_mats, params, n_params}, opt, Spans::ONCE, &c);
        return rc ? rc : emulate(n, c, reinterpret_cast<cd *>(psi), nullptr);
    } catch (const std::bad_alloc &) {
        return QSIM_E_NOMEM;
    }
}

int qsim_debug_emulate_batch(int n, int dtype, const qsim_gate *g, size_t ng, const double *mats, size_t n_mats,
                             const double *params, size_t n_params, const double *uniforms, const int32_t *forced,
                             int n_slots, int max_params, const qsim_fuse_opts *opt, double *psi, int32_t *outcomes,
                             double *probs, int32_t *status) {
    if (n < 1 || n > 24 || (dtype != QSIM_C64 && dtype != QSIM_C128) || (ng && !g) || !psi || !status || n_slots < 0)
        return QSIM_E_ARG;
    for (size_t i = 0; i < ng; i++) {
        if ((g[i].kind == QSIM_G_MEASURE || g[i].kind == QSIM_G_ASSERT0) && (g[i].slot < 0 || g[i].slot >= n_slots))
            return QSIM_E_ARG;
        if (g[i].kind == QSIM_G_MEASURE && !uniforms) return QSIM_E_ARG;
    }
    try {
        Compiled c;
        const bool param = params && n_params;
        int rc = compile_program(n, dtype, g, ng, GateInputs{mats, n_mats, nullptr, param ? n_params : 0}, param, true,
                                 max_params > 0 ? max_params : 2, opt, Spans::REPLAY, &c);
        if (rc) return rc;
        std::vector<qk::BindEntry> ents;
        size_t ncoef = c.plan.coefs.size();
        uint32_t most = 0;
        if (param && (rc = bind_layout(&c, &ents, &ncoef, &most))) return rc;
        if ((rc = validate_plan(n, dtype, c))) return rc;
        if (param) bind_coefs(&c, ents, params, dtype == QSIM_C64, ncoef);
        cd *st = reinterpret_cast<cd *>(psi);
        for (uint64_t x = 0; x < (uint64_t(1) << n); x++) st[x] = x == 0 ? 1.0 : 0.0;
        Records recs;
        recs.uniforms = uniforms;
        recs.forced = forced;
        recs.outcomes = outcomes;
        recs.probs = probs;
        rc = emulate(n, c, st, &recs);
        *status = recs.status;
        return rc;
    } catch (const std::bad_alloc &) {
        return QSIM_E_NOMEM;
    }
}

}  // extern "C"
