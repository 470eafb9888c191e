// C ABI of the simulator (include/qsim.h): state handles, the compile ->
// upload -> launch path of qsim_apply, and the measurement / observable
// calls.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include <new>

#include "host.h"
#include "launch.h"
#include "runtime.h"
#include "swizzle.h"

using namespace qs;

namespace {
thread_local char g_last_error[256] = "";
}

namespace qk {
int note_hip(hipError_t e, const char *where) {
    if (e == hipSuccess) return QSIM_OK;
    std::snprintf(g_last_error, sizeof(g_last_error), "%s: %s (%d)", where, hipGetErrorString(e), int(e));
    return QSIM_E_HIP;
}
}  // namespace qk

namespace qs {

std::atomic<int> g_alloc_countdown{-1};

bool alloc_fault() {
    int v = g_alloc_countdown.load();
    while (v >= 0) {
        if (g_alloc_countdown.compare_exchange_weak(v, v - 1)) return v == 0;
    }
    return false;
}

}  // namespace qs

namespace qs {

size_t elem_bytes(int dtype) { return dtype == QSIM_C64 ? 8 : 16; }

int env_int(const char *name, int dflt) {
    const char *v = std::getenv(name);
    return (v && *v) ? std::atoi(v) : dflt;
}

int resident_max(int dtype) {
    // the whole state in one workgroup's LDS (128 KiB of the 160 KiB)
    return dtype == QSIM_C64 ? 14 : 13;
}

// 12-qubit tiles while a pass gives each CU at most a few of them; complex64
// passes with many tiles (2,048 or more 12-qubit tiles over all the states
// the pass covers: one state of 23+ qubits, or a batch of smaller ones) take
// 13-qubit tiles: several tiles are then queued per CU, so loads, operators
// and stores of different tiles overlap, and the larger tiles carry more
// operators per pass
int default_tile_qubits(int n, int dtype, uint64_t nstates) {
    const bool many = dtype == QSIM_C64 && n > 12 && (nstates << (n - 12)) >= 2048;
    return env_int("QSIM_TILE_QUBITS", many ? 13 : 12);
}

void default_configs(int n, int dtype, const qsim_fuse_opts *opt, FuseConfig *fc, PlanConfig *pc) {
    fc->level = 5;
    fc->max_width = 4;
    fc->sparse = true;
    fc->max_params = 0;
    pc->one_op_per_pass = false;
    pc->tile_qubits = default_tile_qubits(n, dtype, 1);
    pc->low_qubits = env_int("QSIM_LOW_QUBITS", dtype == QSIM_C64 ? 4 : 3);
    pc->window = env_int("QSIM_PLAN_WINDOW", 1024);
    pc->max_tile_k = 4;
    // complex64 tiles use 512 threads; complex128 tiles 256, whose groups of
    // 16 outputs then fit the registers without chunking
    pc->threads = env_int("QSIM_TILE_THREADS", dtype == QSIM_C64 ? 512 : 256) == 256 ? 256 : 512;
    pc->first_in_regs = env_int("QSIM_FIRST_IN_REGS", 1) != 0;
    pc->reg_engine = env_int("QSIM_REG_ENGINE", 0) != 0;
    pc->reg_coalesce = env_int("QSIM_REG_COALESCE", 1) != 0;
    pc->xcd_order = env_int("QSIM_XCD_ORDER", 1) != 0;
    if (opt) {
        if (opt->level >= 0 && opt->level <= 5) fc->level = opt->level;
        if (opt->max_width > 0) fc->max_width = opt->max_width;
        if (opt->tile_qubits > 0) pc->tile_qubits = opt->tile_qubits;
        if (opt->low_qubits > 0) pc->low_qubits = opt->low_qubits;
        pc->one_op_per_pass = (opt->flags & QSIM_F_ONE_OP_PER_PASS) != 0;
        fc->sparse = (opt->flags & QSIM_F_NO_SPARSE) == 0;
        pc->full_support = (opt->flags & QSIM_F_FULL_SUPPORT) != 0;
        if (opt->flags & QSIM_F_REG_ENGINE) pc->reg_engine = true;
    }
    if (dtype == QSIM_C128) fc->max_width = std::min(fc->max_width, 4);
    fc->max_width = std::max(1, std::min(fc->max_width, kMaxK));
    fc->lds_cost = pc->one_op_per_pass ? 64.0 : 3.0;
    if (const char *v = std::getenv("QSIM_LDS_COST")) fc->lds_cost = std::atof(v);
    if (opt && opt->op_cost > 0.0f) fc->lds_cost = opt->op_cost;
    if (!opt || opt->max_width <= 0) fc->max_width = env_int("QSIM_MAX_WIDTH", fc->max_width);
    if (dtype == QSIM_C128) fc->max_width = std::min(fc->max_width, 4);
    fc->max_width = std::max(1, std::min(fc->max_width, kMaxK));
    pc->tile_qubits = std::max(6, std::min(pc->tile_qubits, resident_max(dtype)));
    if (n <= resident_max(dtype)) pc->tile_qubits = n;
    if (pc->tile_qubits > n) pc->tile_qubits = n;
    pc->low_qubits = std::max(0, std::min(pc->low_qubits, pc->tile_qubits - 1));
    // LDS behind the tile (and its reduction scratch) for a pass's records and
    // coefficients: as much as fits without lowering the number of workgroups
    // a CU holds at once, which the tile's LDS and the tile kernel's
    // registers set (two workgroups; four for complex64 tiles of 256
    // threads).  QSIM_META_BUDGET caps it.
    const size_t tile_bytes = (size_t(1) << pc->tile_qubits) * elem_bytes(dtype) + qk::kTileRedBytes;
    const size_t lds = qk::max_lds_bytes();
    const size_t by_regs = (dtype == QSIM_C64 && pc->threads == 256) ? 4 : 2;
    const size_t per_cu = std::max<size_t>(1, std::min(tile_bytes <= lds ? lds / tile_bytes : 0, by_regs));
    const size_t room = lds / per_cu > tile_bytes ? lds / per_cu - tile_bytes : 0;
    pc->meta_budget = std::min(room, size_t(std::max(1024, env_int("QSIM_META_BUDGET", 1 << 30))));
}

// The XCD-order qubits of a tiled pass: distinct qubits outside the tile.
bool xcd_ok(uint64_t rest, int nx, const uint8_t *xq) {
    if (nx < 0 || nx > 3 || nx > __builtin_popcountll(rest)) return false;
    uint64_t seen = 0;
    for (int j = 0; j < nx; j++) {
        if (xq[j] >= 64 || !((rest >> xq[j]) & 1) || ((seen >> xq[j]) & 1)) return false;
        seen |= uint64_t(1) << xq[j];
    }
    return true;
}

// A register-resident pass: tile qubits partition the n qubits, layouts are
// permutations of the tile positions, every record is well formed, the
// re-layout records name the layout the swaps and re-layouts before them
// leave (so the kernel's LDS writes are a permutation of the tile), and
// coefficient ranges lie inside the pass's share of the table.
int validate_reg_pass(int n, int dtype, const Compiled &c, size_t i) {
    const PackedPlan &p = c.plan;
    const PassInfo &pi = c.passes[i];
    const qk::RegArgs &ra = pi.ra;
    const int t = ra.t;
    const uint64_t all = (n >= 64) ? ~uint64_t(0) : ((uint64_t(1) << n) - 1);
    if (pi.strided || pi.kind != Pass::TILE || ra.n != n || reg_threads_for(t) == 0 || t >= n || n - t > 31)
        return QSIM_E_ARG;
    const uint32_t nrec = p.pass_begin[i + 1] - p.pass_begin[i];
    bool any_xpose = false;
    for (uint32_t j = p.pass_begin[i]; j < p.pass_begin[i + 1] && j < p.ops.size(); j++)
        any_xpose |= p.ops[j].kind == DEVOP_XPOSE;
    if (size_t(ra.lds_bytes) != qk::reg_lds_bytes(elem_bytes(dtype), t, any_xpose, nrec) ||
        ra.lds_bytes > qk::max_lds_bytes())
        return QSIM_E_ARG;
    if (ra.flags & ~uint32_t(qk::RF_NONTEMPORAL)) return QSIM_E_ARG;
    uint64_t tile = 0;
    for (int j = 0; j < t; j++) {
        if (ra.tq[j] >= n || (j && ra.tq[j] <= ra.tq[j - 1])) return QSIM_E_ARG;
        tile |= uint64_t(1) << ra.tq[j];
    }
    if ((tile & ra.rest_mask) || ((tile | ra.rest_mask) != all)) return QSIM_E_ARG;
    if (!xcd_ok(ra.rest_mask, ra.nxcd, ra.xcd_q)) return QSIM_E_ARG;
    auto is_perm = [&](const uint8_t *pos) {
        uint32_t seen = 0;
        for (int x = 0; x < t; x++) {
            if (pos[x] >= t || ((seen >> pos[x]) & 1)) return false;
            seen |= 1u << pos[x];
        }
        return true;
    };
    if (!is_perm(ra.load_pos) || !is_perm(ra.store_pos)) return QSIM_E_ARG;
    const uint32_t rb = p.pass_begin[i], re = p.pass_begin[i + 1];
    if (rb > re || re > p.ops.size() || p.coef_begin[i] > p.coef_begin[i + 1] ||
        p.coef_begin[i + 1] > p.coefs.size())
        return QSIM_E_ARG;
    const int logt = t - kRegBits;
    uint8_t cur[16];
    std::memcpy(cur, ra.load_pos, 16);
    for (uint32_t j = rb; j < re; j++) {
        const DevOp &o = p.ops[j];
        if (o.kind == DEVOP_RMAT) {
            if (o.k != kRegBits || o.kx > kMaxK || !o.present || (o.present >> (1 << kRegBits))) return QSIM_E_ARG;
            for (int a = 0; a < o.kx; a++) {
                if (o.xq[a] >= n || ((tile >> o.xq[a]) & 1)) return QSIM_E_ARG;
                if (a && o.xq[a] <= o.xq[a - 1]) return QSIM_E_ARG;
            }
            if (p.op_np[j] < 0 || p.op_np[j] > 3) return QSIM_E_ARG;
            const size_t need = size_t(o.coef) + size_t(devop_coefs(o)) * (size_t(1) << p.op_np[j]);
            if (o.coef < p.coef_begin[i] || need > p.coef_begin[i + 1]) return QSIM_E_ARG;
        } else if (o.kind == DEVOP_SWAP) {
            if ((o.pos[0] != 4 && o.pos[0] != 5) || o.pos[1] >= kRegBits) return QSIM_E_ARG;
            std::swap(cur[o.pos[0]], cur[logt + o.pos[1]]);
        } else if (o.kind == DEVOP_XPOSE) {
            if (j + 1 >= re || p.ops[j + 1].kind != DEVOP_XPOSE2) return QSIM_E_ARG;
            const uint8_t *from = reinterpret_cast<const uint8_t *>(&o);
            const uint8_t *to = reinterpret_cast<const uint8_t *>(&p.ops[j + 1]);
            if (!is_perm(from) || !is_perm(to) || std::memcmp(from, cur, size_t(t)) != 0) return QSIM_E_ARG;
            std::memcpy(cur, to, size_t(t));
            j++;
        } else {
            return QSIM_E_ARG;
        }
    }
    if (std::memcmp(cur, ra.store_pos, size_t(t)) != 0) return QSIM_E_ARG;
    return QSIM_OK;
}

// A span pass: the load vectors and the rest bits generate the index space,
// the store vectors span the same tile, every layout is a bijection onto the
// tile's LDS slots, and masks and coefficients lie inside their ranges.
int validate_span_pass(int n, int dtype, const Compiled &c, size_t i) {
    const PackedPlan &p = c.plan;
    const qk::SpanArgs &sa = c.passes[i].sa;
    const int t = sa.t, logt = t - kSpanRegs;
    const uint64_t all = (uint64_t(1) << n) - 1;
    if (!span_tile_ok(t) || sa.n != n || t > n || n - t > 31 || (sa.rest_mask & ~all) ||
        __builtin_popcountll(sa.rest_mask) != n - t)
        return QSIM_E_ARG;
    // rank of vectors by elimination; `room`: 64 entries, empty at first
    auto add = [](uint64_t *room, uint64_t x) {
        while (x) {
            const int b = 63 - __builtin_clzll(x);
            if (!room[b]) {
                room[b] = x;
                return true;
            }
            x ^= room[b];
        }
        return false;
    };
    uint64_t load[64] = {0}, tile[64] = {0};
    for (int q = 0; q < n; q++)
        if ((sa.rest_mask >> q) & 1) add(load, uint64_t(1) << q);
    for (int j = 0; j < t; j++) {
        if ((sa.load_v[j] & ~all) || (sa.store_v[j] & ~all)) return QSIM_E_ARG;
        if (!add(load, sa.load_v[j]) || !add(tile, sa.load_v[j])) return QSIM_E_ARG;
    }
    uint64_t store[64] = {0};
    for (int j = 0; j < t; j++) {
        if (!add(store, sa.store_v[j])) return QSIM_E_ARG;
        if (add(tile, sa.store_v[j])) return QSIM_E_ARG;   // outside the tile
    }
    const uint32_t rb = p.pass_begin[i], re = p.pass_begin[i + 1];
    if (rb >= re || re > p.ops.size() || p.coef_begin[i] > p.coef_begin[i + 1] ||
        p.coef_begin[i + 1] > p.coefs.size() || p.coef_begin[i + 1] - p.coef_begin[i] < 2 * (re - rb))
        return QSIM_E_ARG;
    if (sa.nrun == 0 || sa.nrun > re - rb || (sa.store_base & ~all) || (sa.store_base && t != n)) return QSIM_E_ARG;
    uint32_t stages = 0, layouts = 0, records = 0, pairs = 0;
    for (uint32_t j = rb; j < re; j++) {
        const DevOp &o = p.ops[j];
        // layouts are numbered as the stages, then the records behind them
        if ((o.kind == DEVOP_LAYOUT) != (j - rb >= sa.nrun)) return QSIM_E_ARG;
        if (o.kind == DEVOP_STAGE || o.kind == DEVOP_LAYOUT) {
            const uint8_t *raw = reinterpret_cast<const uint8_t *>(&o);
            uint64_t slots[64] = {0};
            if (o.kx != layouts || layouts >= 255 || (o.kind == DEVOP_LAYOUT && t != n)) return QSIM_E_ARG;
            for (int x = 0; x < t; x++) {
                uint16_t s;
                std::memcpy(&s, raw + (x < 7 ? 2 * x : 16 + 2 * (x - 7)), 2);
                if ((s >> t) || !add(slots, s)) return QSIM_E_ARG;
            }
            uint16_t c;
            std::memcpy(&c, raw + 30, 2);
            if (c >> t || (c && o.kind == DEVOP_STAGE)) return QSIM_E_ARG;
            layouts++;
            if (o.kind == DEVOP_STAGE) stages++;
        } else if (o.kind == DEVOP_SPAN_REC) {
            // each has a layout of its own, in order, behind the stages
            if (!stages || t != n || !devop_is_record(o.pos[0]) || (o.slot[0] >> logt) || (o.present >> 8) ||
                ((o.present >> 4) & 7) > kSpanRegs || p.op_np[j] != 0)
                return QSIM_E_ARG;
            const bool moves = o.pos[0] == DEVOP_RESET || o.pos[0] == DEVOP_MEASURE_RESET;
            if (moves && !((o.present >> 4) & 7)) return QSIM_E_ARG;
            records++;
        } else if (o.kind == DEVOP_PAULI) {
            if (!stages || o.k > 2 * kSpanRegs || (o.slot[0] >> logt) ||
                (o.present >> (1 << kSpanRegs)) || p.op_np[j] != 0)
                return QSIM_E_ARG;
            // the kernel finds the coefficients at twice the record's number
            if (o.coef != p.coef_begin[i] + 2 * (j - rb)) return QSIM_E_ARG;
        } else if (o.kind == DEVOP_PAULI2) {
            // and two records behind it; its branch is that of both members of a pair
            if (!stages || o.k >= 2 * kSpanRegs || (o.slot[0] >> logt) || (o.present >> kSpanRegs) || p.op_np[j] != 0 ||
                o.coef != p.coef_begin[i] + 2 * (j - rb) || j - rb + 2 >= sa.nrun)
                return QSIM_E_ARG;
            const DevOp &w = p.ops[j + 1];
            if (w.kind != DEVOP_PAULI2X || p.ops[j + 2].kind != DEVOP_PAULI2X || (w.slot[0] >> logt) ||
                (w.present >> kSpanRegs) || ((w.present >> (o.k >> 1)) & 1) || p.op_np[j + 1] != 0 || p.op_np[j + 2] != 0)
                return QSIM_E_ARG;
            pairs++;
            j += 2;
        } else {
            return QSIM_E_ARG;
        }
    }
    if (p.ops[rb].kind != DEVOP_STAGE || sa.tile_bytes != (stages > 1 ? uint32_t(elem_bytes(dtype) << t) : 0u) ||
        sa.nlayout != layouts || layouts != stages + records || sa.pairs != pairs ||
        qk::span_lds_bytes(sa.tile_bytes, re - rb, layouts) > qk::max_lds_bytes())
        return QSIM_E_ARG;
    uint32_t at = stages;
    for (uint32_t j = rb; j < re; j++)
        if (p.ops[j].kind == DEVOP_SPAN_REC && p.ops[j].kx != at++) return QSIM_E_ARG;
    return QSIM_OK;
}

// Check, before anything is launched, that every device record stays inside
// the buffers and tiles the kernels will index: tile qubits partition the n
// qubits, operator positions are ascending and inside the tile (or the
// state), and coefficient ranges lie inside the coefficient table.
int validate_plan(int n, int dtype, const Compiled &c) {
    const PackedPlan &p = c.plan;
    if (p.pass_begin.size() != c.passes.size() + 1 || p.coef_begin.size() != c.passes.size() + 1)
        return QSIM_E_ARG;
    const uint64_t all = (n >= 64) ? ~uint64_t(0) : ((uint64_t(1) << n) - 1);
    for (size_t i = 0; i < c.passes.size(); i++) {
        const PassInfo &pi = c.passes[i];
        int width = n;
        if (pi.reg || pi.span) {
            const int rc = pi.reg ? validate_reg_pass(n, dtype, c, i) : validate_span_pass(n, dtype, c, i);
            if (rc) return rc;
            continue;
        }
        if (pi.kind == Pass::MEASURE) {
            if (p.pass_begin[i] != p.pass_begin[i + 1] || pi.meas.q < 0 || pi.meas.q >= n ||
                !devop_is_record(pi.meas.kind))
                return QSIM_E_ARG;
            continue;
        }
        if (!pi.strided) {
            const qk::TileArgs &ta = pi.ta;
            if (ta.n != n || ta.t < 1 || ta.t > n || ta.t > resident_max(dtype) || ta.c < 0 ||
                ta.c > ta.t || ta.nhi != ta.t - ta.c || n - ta.t > 31)
                return QSIM_E_ARG;
            uint64_t m = (uint64_t(1) << ta.c) - 1;
            int prev = ta.c - 1;
            for (int h = 0; h < ta.nhi; h++) {
                if (ta.hi[h] <= prev || ta.hi[h] >= n) return QSIM_E_ARG;
                prev = ta.hi[h];
                m |= uint64_t(1) << ta.hi[h];
            }
            if ((m & ta.rest_mask) || ((m | ta.rest_mask) != all) || m != ta.tile_mask) return QSIM_E_ARG;
            if (!xcd_ok(ta.rest_mask, ta.nxcd, ta.xcd_q)) return QSIM_E_ARG;
            // tile positions: the low qubits first, then every other tile
            // qubit once
            uint64_t mq = 0;
            for (int j = 0; j < ta.t; j++) {
                if (j < ta.c && ta.tq[j] != j) return QSIM_E_ARG;
                if (ta.tq[j] >= n || ((mq >> ta.tq[j]) & 1)) return QSIM_E_ARG;
                mq |= uint64_t(1) << ta.tq[j];
            }
            if (mq != ta.tile_mask) return QSIM_E_ARG;
            if (ta.regs) {
                // operators run on a thread's registers: their tile positions
                // are consecutive register-index bits (log2(threads) + off + j)
                const int logt = ta.threads == 512 ? 9 : 8;
                const uint32_t rb = p.pass_begin[i], re = p.pass_begin[i + 1];
                const int first = ta.regs & 1, last = (ta.regs >> 1) & 1, off = (ta.regs >> 2) & 7;
                if ((ta.regs >> 5) || ta.t <= logt || ta.t >= n || re - rb < uint32_t(first + last)) return QSIM_E_ARG;
                const int le = std::min(ta.t - logt, 4);
                auto check_regs = [&](const DevOp &o, int at) {
                    if (o.kind != DEVOP_MAT || o.k > first_regs_max_k(dtype) || at + o.k > le) return false;
                    for (int a2 = 0; a2 < o.k; a2++)
                        if (o.pos[a2] != logt + at + a2) return false;
                    return true;
                };
                if (first && !check_regs(p.ops[rb], 0)) return QSIM_E_ARG;
                if (last && (!check_regs(p.ops[re - 1], off) || off != (first ? int(p.ops[rb].k) : 0)))
                    return QSIM_E_ARG;
                if (!last && off) return QSIM_E_ARG;
            }
            width = ta.t;
        }
        if (p.pass_begin[i] > p.pass_begin[i + 1] || p.pass_begin[i + 1] > p.ops.size()) return QSIM_E_ARG;
        if (p.coef_begin[i] > p.coef_begin[i + 1] || p.coef_begin[i + 1] > p.coefs.size()) return QSIM_E_ARG;
        if (!pi.strided &&
            qk::tile_lds_bytes(elem_bytes(dtype), pi.ta.t, p.pass_begin[i + 1] - p.pass_begin[i],
                               p.coef_begin[i + 1] - p.coef_begin[i]) > qk::max_lds_bytes())
            return QSIM_E_ARG;
        for (uint32_t j = p.pass_begin[i]; j < p.pass_begin[i + 1]; j++) {
            const DevOp &o = p.ops[j];
            if (o.kind == DEVOP_RUN) {
                // 2-qubit operators on four positions, none of them one of those
                // that run on registers at the ends of the pass
                const uint32_t end = p.pass_begin[i + 1] - ((pi.ta.regs >> 1) & 1);
                if (pi.strided || !run_tile(elem_bytes(dtype), width) || o.k != 4 || o.present < 2 || o.present >= end - j ||
                    (j == p.pass_begin[i] && (pi.ta.regs & 1)))
                    return QSIM_E_ARG;
                for (int a = 0; a < 4; a++)
                    if (o.pos[a] >= width || (a && o.pos[a] <= o.pos[a - 1]) ||
                        o.slot[a] != lds_slot(int(elem_bytes(dtype)), 1 << o.pos[a]))
                        return QSIM_E_ARG;
                for (uint32_t x = j + 1; x <= j + o.present; x++) {
                    const DevOp &m = p.ops[x];
                    if (m.kind != DEVOP_MAT || m.k != 2 || m.kx || m.xq[0] > 5 ||
                        m.pos[0] != o.pos[kRunPair[m.xq[0]][0]] || m.pos[1] != o.pos[kRunPair[m.xq[0]][1]])
                        return QSIM_E_ARG;
                }
                continue;
            }
            if (o.kind != DEVOP_MAT) {
                // measurement records run only inside resident (whole-state) passes
                if (pi.strided || pi.ta.t != n || o.pos[0] >= n || !devop_is_record(o.kind)) return QSIM_E_ARG;
                continue;
            }
            // tiled passes may hold operators with block qubits (kx > 0),
            // which must lie outside the tile; k = 0 then is an operator
            // diagonal on all its qubits
            if (pi.strided ? (o.kx != 0 || o.k < 1) : (o.k + o.kx < 1)) return QSIM_E_ARG;
            if (o.k > width || o.k + o.kx > kMaxK) return QSIM_E_ARG;
            if (!pi.strided && o.k > 4) return QSIM_E_ARG;
            for (int a = 0; a < o.k; a++) {
                if (o.pos[a] >= width) return QSIM_E_ARG;
                if (a && o.pos[a] <= o.pos[a - 1]) return QSIM_E_ARG;
                if (!pi.strided && o.slot[a] != lds_slot(int(elem_bytes(dtype)), 1 << o.pos[a])) return QSIM_E_ARG;
            }
            for (int a = 0; a < o.kx; a++) {
                if (o.xq[a] >= n || ((pi.ta.tile_mask >> o.xq[a]) & 1)) return QSIM_E_ARG;
                if (a && o.xq[a] <= o.xq[a - 1]) return QSIM_E_ARG;
            }
            const uint32_t d = 1u << o.k;
            const uint32_t mask = (d >= 32) ? 0xffffffffu : ((1u << d) - 1);
            if (!o.present || (o.present & ~mask)) return QSIM_E_ARG;
            const size_t need = size_t(o.coef) + size_t(devop_coefs(o)) * (size_t(1) << p.op_np[j]);
            if (need > p.coefs.size()) return QSIM_E_ARG;
            if (!pi.strided && (o.coef < p.coef_begin[i] || need > p.coef_begin[i + 1])) return QSIM_E_ARG;
            if (p.op_np[j] < 0 || p.op_np[j] > 3) return QSIM_E_ARG;
        }
    }
    return QSIM_OK;
}

// Whether a circuit may run as a Pauli program (QSIM_SPAN=0 turns it off): with
// level-5 fusion and no option that asks for another form of operator or pass,
// or that keeps commuting operators in order.
// A whole state in one tile is such a pass too, its measurement records inside:
// against k_tile's resident ones, 120 exponentials on 13 qubits complex128 run in
// 67 us (284) and 250 on 14 qubits complex64 in 161 us (493); states below 10
// qubits have too few amplitudes for a wave's registers.
static bool spans_wanted(int n, const FuseConfig &fc, const PlanConfig &pc) {
    return fc.level == 5 && fc.sparse && !pc.one_op_per_pass && !pc.reg_engine && span_tile_ok(pc.tile_qubits) &&
           n - pc.tile_qubits <= 31 &&
           env_int("QSIM_SPAN", 1) != 0 && env_int("QSIM_PLAN_COMMUTE", 1) != 0;
}

// The operators of L, fused, planned and packed into *out.
static int compile_ops(int n, int dtype, Lowered *L, const FuseConfig &fc, const PlanConfig &pc, Compiled *out) {
    int64_t counts[6];
    {
        TraceRange r("qsim.fuse");
        fuse(n, L, fc, counts);
    }
    TraceRange plan_range("qsim.plan");
    std::vector<uint32_t> present(L->ops.size()), meta(L->ops.size());
    for (size_t i = 0; i < L->ops.size(); i++) {
        present[i] = op_present(L->ops[i], fc.sparse);
        // LDS holds the bound (per-state) coefficients: no cos/sin blocks
        meta[i] = uint32_t(sizeof(DevOp) + size_t(__builtin_popcount(present[i])) *
                                               L->ops[i].dim() * elem_bytes(dtype));
    }
    std::vector<uint64_t> need(L->ops.size());
    for (size_t i = 0; i < L->ops.size(); i++)
        need[i] = pc.full_support ? L->ops[i].mask() : op_moved_qubits(L->ops[i], present[i]);
    std::vector<Pass> passes;
    plan_passes(n, *L, meta, need, pc, &passes);
    // tiled passes of 10..13 qubits (not whole-state ones, which may hold
    // measurement records) run register-resident
    for (Pass &p : passes)
        p.reg = pc.reg_engine && p.kind == Pass::TILE && !p.strided && p.t < n && reg_threads_for(p.t) > 0 &&
                p.c <= 4 && p.inline_meas.empty();
    place_positions(n, L->ops, pc.threads == 512 ? 9 : 8, first_regs_max_k(dtype), pc.first_in_regs, &passes);
    if (pc.xcd_order) place_xcd_qubits(n, &passes);
    const int rc = pack_plan(L->ops, present, passes, pc, &out->plan);
    if (rc) return rc;
    group_runs(passes, elem_bytes(dtype), pc.meta_budget, &out->plan);
    // LDS slot offsets of the tile positions (the tile kernel's layout)
    for (size_t i = 0; i < passes.size(); i++) {
        if (passes[i].strided || passes[i].kind != Pass::TILE) continue;
        for (uint32_t j = out->plan.pass_begin[i]; j < out->plan.pass_begin[i + 1]; j++) {
            DevOp &o = out->plan.ops[j];
            if (o.kind != DEVOP_MAT && o.kind != DEVOP_RUN) continue;
            for (int a = 0; a < o.k; a++) o.slot[a] = uint16_t(lds_slot(int(elem_bytes(dtype)), 1 << o.pos[a]));
        }
    }
    out->passes.clear();
    out->passes.reserve(passes.size());
    for (const Pass &p : passes) {
        PassInfo pi;
        pi.kind = p.kind;
        pi.meas = p.meas;
        pi.strided = p.strided;
        pi.ta.n = n;
        pi.ta.t = p.t;
        pi.ta.c = p.c;
        pi.ta.nhi = p.nhi;
        uint64_t all = (n >= 64) ? ~uint64_t(0) : ((uint64_t(1) << n) - 1);
        pi.ta.rest_mask = all & ~p.tile_mask;
        pi.ta.tile_mask = p.tile_mask;
        pi.ta.threads = pc.threads;
        pi.ta.regs = (p.first_in_regs ? 1 : 0) | (p.last_in_regs ? 2 : 0) | (p.last_off << 2);
        for (int h = 0; h < p.nhi; h++) pi.ta.hi[h] = uint8_t(p.hi[h]);
        for (int j = 0; j < 16; j++) pi.ta.tq[j] = p.tq[j];
        pi.ta.nxcd = p.nxcd;
        for (int j = 0; j < 4; j++) pi.ta.xcd_q[j] = p.xcd_q[j];
        if (p.reg) {
            pi.ra.nxcd = p.nxcd;
            for (int j = 0; j < 4; j++) pi.ra.xcd_q[j] = p.xcd_q[j];
            pi.reg = true;
            pi.ra.rest_mask = pi.ta.rest_mask;
            pi.ra.n = n;
            pi.ra.t = p.t;
            pi.ra.lds_bytes = uint32_t(qk::reg_lds_bytes(elem_bytes(dtype), p.t, p.reg_xposes > 0,
                                                         out->plan.pass_begin[out->passes.size() + 1] -
                                                             out->plan.pass_begin[out->passes.size()]));
            // states beyond the 256 MB Infinity Cache stream from HBM:
            // non-temporal loads and stores there
            pi.ra.flags = ((elem_bytes(dtype) << n) > (size_t(256) << 20)) ? qk::RF_NONTEMPORAL : 0u;
            for (int j = 0; j < 16; j++) {
                pi.ra.tq[j] = p.tq[j];
                pi.ra.load_pos[j] = p.load_pos[j];
                pi.ra.store_pos[j] = p.store_pos[j];
            }
            out->stats_reg_swaps += p.reg_swaps;
            out->stats_reg_xposes += p.reg_xposes;
        }
        out->passes.push_back(pi);
    }
    qsim_apply_stats &s = out->stats;
    std::memset(&s, 0, sizeof(s));
    s.input_gates = L->input_gates;
    for (int l = 0; l < 6; l++) s.ops_after[l] = counts[l];
    s.fused_ops = int64_t(L->ops.size());
    out->records = int64_t(L->meas.size());
    s.passes = int64_t(passes.size());
    s.terms = out->plan.terms;
    s.bytes_moved = int64_t(passes.size()) * 2 * (int64_t(1) << n) * int64_t(elem_bytes(dtype));
    s.tile_qubits = pc.one_op_per_pass ? 0 : pc.tile_qubits;
    s.max_width = fc.max_width;
    for (const PassInfo &pi : out->passes) s.reg_passes += pi.reg ? 1 : 0;
    s.reg_swaps = out->stats_reg_swaps;
    s.reg_relayouts = out->stats_reg_xposes;
    return QSIM_OK;
}

// The passes of `src` behind those of *out, whose ends are still open.
static void append_passes(const Compiled &src, Compiled *out) {
    const PackedPlan &s = src.plan;
    PackedPlan &p = out->plan;
    const uint32_t o0 = uint32_t(p.ops.size()), c0 = uint32_t(p.coefs.size());
    for (size_t i = 0; i < src.passes.size(); i++) {
        out->passes.push_back(src.passes[i]);
        p.pass_begin.push_back(o0 + s.pass_begin[i]);
        p.coef_begin.push_back(c0 + s.coef_begin[i]);
    }
    for (DevOp o : s.ops) {
        if (devop_has_place(o.kind)) o.coef += c0;
        p.ops.push_back(o);
    }
    p.coefs.insert(p.coefs.end(), s.coefs.begin(), s.coefs.end());
    p.op_np.insert(p.op_np.end(), s.op_np.begin(), s.op_np.end());
    p.op_slots.insert(p.op_slots.end(), s.op_slots.begin(), s.op_slots.end());
    p.terms += s.terms;
}

// The plan of a Pauli program, with the measurement records of L.
static int compile_spans(int n, int dtype, const PauliProgram &P, const Lowered &L, const FuseConfig &fc,
                         const PlanConfig &pc, Compiled *out) {
    TraceRange range("qsim.plan");
    const size_t elem = elem_bytes(dtype);
    const int t = pc.tile_qubits;
    const bool whole = t == n;
    PackedPlan &pl = out->plan;
    const uint64_t all = (uint64_t(1) << n) - 1;
    bool phased = P.phase == 0.0;
    size_t left_ops = 0;
    auto put = [&](const Pass &p, bool last) -> int {
        pl.pass_begin.push_back(uint32_t(pl.ops.size()));
        pl.coef_begin.push_back(uint32_t(pl.coefs.size()));
        PassInfo pi;
        pi.kind = p.kind;
        pi.meas = p.meas;
        if (p.span) {
            qk::SpanArgs &sa = pi.sa;
            const int rc = pack_span_pass(P, p, kSpanRegs, dtype == QSIM_C64, &pl, &sa.nrun);
            if (rc) return rc;
            pi.span = true;
            pi.ta.n = n;
            sa.n = n;
            sa.t = p.t;
            sa.rest_mask = all & ~p.tile_mask;
            for (int j = 0; j < p.t; j++) {
                sa.load_v[j] = span_vector(p, p.stages.front().layout[j]);
                sa.store_v[j] = span_vector(p, p.stages.back().layout[j]);
                if (last) sa.store_v[j] = map_index(P.map, sa.store_v[j]);
            }
            if (last) sa.store_base = P.map.c;
            sa.tile_bytes = p.stages.size() > 1 ? uint32_t(elem << p.t) : 0u;
            sa.nlayout = uint32_t(p.stages.size() + (pl.ops.size() - pl.pass_begin.back() - sa.nrun));
            for (uint32_t j = pl.pass_begin.back(); j < pl.ops.size(); j++) sa.pairs += pl.ops[j].kind == DEVOP_PAULI2;
            sa.phase_re = 1.0;
            if (!phased) {
                sa.phase_re = std::cos(P.phase);
                sa.phase_im = std::sin(P.phase);
                phased = true;
            }
        }
        out->passes.push_back(pi);
        return QSIM_OK;
    };
    // the gates that epoch e leaves in the frame
    size_t left_at = 0;
    auto put_left = [&](int e) -> int {
        size_t end = left_at;
        while (end < P.left.size() && P.left_epoch[end] == e) end++;
        if (end == left_at) return QSIM_OK;
        Lowered T;
        int rc = lower(n, P.left.data() + left_at, end - left_at, GateInputs{}, false, false, &T);
        left_at = end;
        Compiled c;
        if (!rc) rc = compile_ops(n, dtype, &T, fc, pc, &c);
        if (!rc) append_passes(c, out);
        left_ops += T.ops.size();
        return rc;
    };
    std::vector<Pass> passes;
    int rc = QSIM_OK;
    // for a pass without rotations, where only a permutation or a phase is left
    auto identity = [] {
        PauliProgram none;
        none.ops.push_back(PauliOp{});
        none.op_epoch.push_back(0);
        return none;
    };
    if (whole) {
        plan_whole(n, P, L.n_epochs, pc.low_qubits, kSpanRegs, pc.meta_budget, &passes);
        if (passes.empty() && (!P.map.z.empty() || !phased)) {
            plan_whole(n, identity(), 0, pc.low_qubits, kSpanRegs, pc.meta_budget, &passes);
            passes[0].stages[0].ops.clear();
        }
        for (size_t i = 0; i < passes.size() && !rc; i++) rc = put(passes[i], i + 1 == passes.size());
        if (!rc) rc = put_left(L.n_epochs);   // (follows every record)
    } else {
        size_t at = 0, m = 0;
        if (P.ops.empty() && !phased) {
            plan_spans(n, identity(), t, pc.low_qubits, kSpanRegs, pc.meta_budget, pc.window, false, 0, 1, &passes);
            passes[0].stages[0].ops.clear();
            rc = put(passes[0], false);
        }
        for (int e = 0; e < L.n_epochs && !rc; e++) {
            size_t end = at;
            while (end < P.ops.size() && P.op_epoch[end] == e) end++;
            passes.clear();
            plan_spans(n, P, t, pc.low_qubits, kSpanRegs, pc.meta_budget, pc.window, pc.full_support, int(at),
                       int(end), &passes);
            at = end;
            for (size_t i = 0; i < passes.size() && !rc; i++) rc = put(passes[i], false);
            if (!rc) rc = put_left(e);
            for (; m < L.meas.size() && L.meas[m].epoch == e && !rc; m++) {
                Pass p;
                p.kind = Pass::MEASURE;
                p.meas = L.meas[m];
                rc = put(p, false);
            }
        }
    }
    if (rc) return rc;
    out->pauli = true;
    pl.pass_begin.push_back(uint32_t(pl.ops.size()));
    pl.coef_begin.push_back(uint32_t(pl.coefs.size()));
    out->records = int64_t(L.meas.size());
    qsim_apply_stats &s = out->stats;
    std::memset(&s, 0, sizeof(s));
    s.input_gates = L.input_gates;
    for (int l = 1; l < 5; l++) s.ops_after[l] = -1;   // the paper's fusion steps are not taken
    s.ops_after[0] = L.input_gates;
    s.ops_after[5] = s.fused_ops = int64_t(P.ops.size() + left_ops);
    s.passes = int64_t(out->passes.size());
    s.terms = pl.terms;
    for (const DevOp &o : pl.ops) s.reg_relayouts += o.kind == DEVOP_STAGE ? 1 : 0;
    for (const PassInfo &pi : out->passes) s.reg_relayouts -= pi.span ? 1 : 0;
    s.bytes_moved = s.passes * 2 * (int64_t(1) << n) * int64_t(elem);
    s.tile_qubits = t;
    return QSIM_OK;
}

// Modelled run time of a plan, in the time of a rotation in k_span.  Fitted to 12
// families of circuits (QFT, layers of rotations, Trotter steps, QAOA, random
// rotations, Pauli exponentials) at 10 to 30 qubits in both types, single states:
// within 10% of most times, 25% of all; taking the cheaper plan by it costs 1% of
// the better one's time on average, 23% at worst (53 us for 44).  184 batches of 8
// to 512 states, 72 of them with angles per state: 1% on average, at worst 78 us for
// 65 (exchange layers at 10 qubits complex64) and 385 for 329 (a QFT at 14 qubits
// complex128).
static double plan_cost(const Compiled &c, int dtype) {
    const bool single = dtype == QSIM_C64;
    double cost = 0.0;
    for (size_t i = 0; i < c.passes.size(); i++) {
        if (c.passes[i].kind == Pass::MEASURE) continue;   // the same in every plan
        // (the passes of gates left in the frame as those of rotations)
        cost += c.pauli ? (single ? 26.0 : 32.0) : (single ? 14.0 : 18.0);
        for (uint32_t j = c.plan.pass_begin[i]; j < c.plan.pass_begin[i + 1]; j++) {
            const DevOp &o = c.plan.ops[j];
            if (o.kind == DEVOP_STAGE) cost += 1.5;
            else if (o.kind == DEVOP_PAULI) cost += 1.0;
            else if (o.kind == DEVOP_PAULI2) cost += 2.0;
            else if (o.kind == DEVOP_MAT && !c.pauli)
                cost += (single ? 4.0 : 5.5) + (single ? 0.7 : 1.1) * __builtin_popcount(o.present);
        }
    }
    return cost;
}

// Whether the tiled plan of a circuit is worth the compile beside its span passes.
// Fused operators gain where gates share qubits and each is a rotation of its own:
// Pauli exponentials written with CX are a rotation per 3 gates and more.  A
// circuit that runs once saves less than half of its span passes' time, about a
// fifth where it saves any, for at least 100 us + 1.5 us a gate of compile time; a
// rotation takes 0.3 us, and beyond 16 MiB about 8 ns per MiB of the state.
// QSIM_SPAN=2 takes span passes wherever they are possible.
static bool spans_may_lose(int n, int dtype, const PauliProgram &P, const Lowered &L, const PlanConfig &pc, Spans spans,
                           const Compiled &c) {
    if (env_int("QSIM_SPAN", 1) >= 2) return false;
    size_t rots = 0;
    for (const PauliOp &o : P.ops) rots += o.two ? 2 : 1;
    if (double(rots) <= 0.35 * double(L.input_gates)) return false;
    if (spans == Spans::ONCE) {
        const double us = plan_cost(c, dtype) * (0.3 + 8e-9 * std::ldexp(double(elem_bytes(dtype)), n));
        return us > 3.0 * (100.0 + 1.5 * double(L.input_gates));
    }
    return true;
}

int compile_circuit(int n, int dtype, const qsim_gate *g, size_t ng, const GateInputs &in,
                    const qsim_fuse_opts *opt, Spans spans, Compiled *out) {
    return compile_program(n, dtype, g, ng, in, false, false, 0, opt, spans, out);
}

int compile_program(int n, int dtype, const qsim_gate *g, size_t ng, const GateInputs &in,
                    bool keep_params, bool allow_meas, int max_params,
                    const qsim_fuse_opts *opt, Spans spans, Compiled *out) {
    TraceRange range("qsim.compile");
    double t0 = now_seconds();
    if (alloc_fault()) throw std::bad_alloc();
    FuseConfig fc;
    PlanConfig pc;
    default_configs(n, dtype, opt, &fc, &pc);
    fc.max_params = keep_params ? std::max(1, std::min(max_params, 3)) : 0;
    Lowered L;
    int rc;
    Compiled rotations;   // the plan of span passes, if there is one
    {
        TraceRange r("qsim.lower");
        std::vector<size_t> op_gate;
        size_t first_at;
        split_records(n, g, ng, allow_meas, &L, &op_gate, &rc, &first_at);
        if (!rc && spans != Spans::OFF && spans_wanted(n, fc, pc)) {
            PauliProgram P;
            bool fits = pauli_lower(n, g, op_gate, L, in, keep_params, pc.tile_qubits == n, &P);
            if (pc.full_support)
                for (const PauliOp &o : P.ops)
                    fits = fits && __builtin_popcountll(o.x | o.z | o.z2) <= pc.tile_qubits - pc.low_qubits;
            if (fits) {
                rc = compile_spans(n, dtype, P, L, fc, pc, &rotations);
                if (rc) return rc;
                rotations.stats.max_width = fc.max_width;
                if (!spans_may_lose(n, dtype, P, L, pc, spans, rotations)) {
                    *out = std::move(rotations);
                    out->fixed = true;
                    out->stats.compile_seconds = now_seconds() - t0;
                    return keep_params ? QSIM_OK : validate_plan(n, dtype, *out);
                }
            }
        }
        rc = lower_gates(n, g, ng, in, keep_params, op_gate, rc, first_at, &L);
    }
    if (rc) return rc;
    rc = compile_ops(n, dtype, &L, fc, pc, out);
    if (rc) return rc;
    if (rotations.pauli && plan_cost(rotations, dtype) < plan_cost(*out, dtype)) *out = std::move(rotations);
    qsim_apply_stats &s = out->stats;
    s.compile_seconds = now_seconds() - t0;
    // parameterised templates are validated after their coefficient layout
    // is bound (qsim_batch_create)
    return keep_params ? QSIM_OK : validate_plan(n, dtype, *out);
}

}  // namespace qs

// ------------------------------------------------------------- handles
namespace {

int hip_rc(hipError_t e) { return qk::note_hip(e, "runtime call"); }

int grow(void **ptr, size_t *cap, size_t need, hipStream_t st) {
    if (need <= *cap) return QSIM_OK;
    if (qs::alloc_fault()) return QSIM_E_NOMEM;   // before anything is freed
    if (*ptr) {
        (void)hipStreamSynchronize(st);
        (void)hipFree(*ptr);
        *ptr = nullptr;
        *cap = 0;
    }
    size_t sz = std::max(need, size_t(4096));
    sz = (sz + sz / 4 + 255) & ~size_t(255);
    hipError_t e = hipMalloc(ptr, sz);
    if (e != hipSuccess) { qk::note_hip(e, "hipMalloc"); *ptr = nullptr; return QSIM_E_NOMEM; }
    *cap = sz;
    return QSIM_OK;
}

int grow_host(void **ptr, size_t *cap, size_t need) {
    if (need <= *cap) return QSIM_OK;
    if (qs::alloc_fault()) return QSIM_E_NOMEM;
    if (*ptr) (void)hipHostFree(*ptr);
    *ptr = nullptr;
    *cap = 0;
    size_t sz = std::max(need, size_t(1) << 17);   // (freeing one to grow it waits for the device)
    sz = (sz + sz / 4 + 255) & ~size_t(255);
    hipError_t e = hipHostMalloc(ptr, sz, hipHostMallocDefault);
    if (e != hipSuccess) { qk::note_hip(e, "hipHostMalloc"); *ptr = nullptr; return QSIM_E_NOMEM; }
    *cap = sz;
    return QSIM_OK;
}

}  // namespace

namespace qs {

// Copy the packed plan to pinned staging (coefficients cast to the state
// precision) and then to the device, asynchronously on `st`.
int upload_plan(DeviceTables *dt, int dtype, const PackedPlan &plan, hipStream_t st) {
    const size_t ops_bytes = plan.ops.size() * sizeof(DevOp);
    const size_t coef_bytes = plan.coefs.size() * elem_bytes(dtype);
    const size_t ops_pad = (ops_bytes + 255) & ~size_t(255);
    if (dt->stage_ev_valid) {
        (void)hipEventSynchronize(dt->stage_ev);   // previous upload has left the staging buffer
        dt->stage_ev_valid = false;
    }
    int rc = grow_host(&dt->h_stage, &dt->cap_stage, ops_pad + coef_bytes + 256);
    if (rc) return rc;
    rc = grow((void **)&dt->d_ops, &dt->cap_ops, ops_pad + 256, st);
    if (rc) return rc;
    rc = grow(&dt->d_coefs, &dt->cap_coefs, coef_bytes + 256, st);
    if (rc) return rc;
    unsigned char *h = (unsigned char *)dt->h_stage;
    if (ops_bytes) std::memcpy(h, plan.ops.data(), ops_bytes);
    if (dtype == QSIM_C64) {
        float *c = (float *)(h + ops_pad);
        for (size_t i = 0; i < plan.coefs.size(); i++) {
            c[2 * i] = float(plan.coefs[i].real());
            c[2 * i + 1] = float(plan.coefs[i].imag());
        }
    } else if (coef_bytes) {
        std::memcpy(h + ops_pad, plan.coefs.data(), coef_bytes);
    }
    if (ops_bytes && hipMemcpyAsync(dt->d_ops, h, ops_bytes, hipMemcpyHostToDevice, st) != hipSuccess)
        return QSIM_E_HIP;
    if (coef_bytes &&
        hipMemcpyAsync(dt->d_coefs, h + ops_pad, coef_bytes, hipMemcpyHostToDevice, st) != hipSuccess)
        return QSIM_E_HIP;
    if (!dt->stage_ev) {
        if (hipEventCreateWithFlags(&dt->stage_ev, hipEventDisableTiming) != hipSuccess) return QSIM_E_HIP;
    }
    if (hipEventRecord(dt->stage_ev, st) != hipSuccess) return QSIM_E_HIP;
    dt->stage_ev_valid = true;
    return QSIM_OK;
}

void free_tables(DeviceTables *dt) {
    if (dt->stage_ev_valid) (void)hipEventSynchronize(dt->stage_ev);
    if (dt->stage_ev) (void)hipEventDestroy(dt->stage_ev);
    if (dt->d_ops) (void)hipFree(dt->d_ops);
    if (dt->d_coefs) (void)hipFree(dt->d_coefs);
    if (dt->h_stage) (void)hipHostFree(dt->h_stage);
    *dt = DeviceTables{};
}

int enqueue_pass(const Compiled &c, size_t i, const DevOp *d_ops, const void *d_coefs, uint64_t cstride, int dtype,
                 void *state, uint64_t sstride, uint32_t nstates, const qk::MeasArgs *ma, uint32_t flags,
                 hipStream_t st) {
    const PackedPlan &p = c.plan;
    const PassInfo &pi = c.passes[i];
    const uint32_t ob = p.pass_begin[i], oe = p.pass_begin[i + 1], cb = p.coef_begin[i], ce = p.coef_begin[i + 1];
    const int32_t *status = ma ? ma->status : nullptr;
    if (pi.kind == Pass::MEASURE) return QSIM_E_UNSUPPORTED;
    if (pi.strided) {
        for (uint32_t j = ob; j < oe; j++) {
            const int rc =
                qk::launch_sweep(dtype, state, sstride, nstates, pi.ta.n, p.ops[j], d_coefs, st, cstride, status);
            if (rc) return rc;
        }
        return QSIM_OK;
    }
    if (pi.span)
        return qk::launch_span(dtype, state, sstride, nstates, pi.sa, d_ops, ob, oe, d_coefs, cb, cstride,
                               ma ? *ma : qk::MeasArgs{}, flags, st);
    if (pi.reg)
        return qk::launch_reg(dtype, state, sstride, nstates, pi.ra, d_ops, ob, oe, d_coefs, cb, ce, cstride, status,
                              flags, st);
    return qk::launch_tile(dtype, state, sstride, nstates, pi.ta, d_ops, ob, oe, d_coefs, cb, ce, cstride, ma, flags,
                           st);
}

int enqueue_passes(const Compiled &c, const DeviceTables &dt, int dtype, void *state,
                   hipStream_t st, bool init_zero_first, uint64_t sstride, uint32_t nstates) {
    for (size_t i = 0; i < c.passes.size(); i++) {
        const uint32_t flags = (init_zero_first && i == 0) ? qk::TF_INIT_ZERO : 0u;
        const int rc =
            enqueue_pass(c, i, dt.d_ops, dt.d_coefs, 0, dtype, state, sstride, nstates, nullptr, flags, st);
        if (rc) return rc;
    }
    return QSIM_OK;
}

}  // namespace qs

struct qsim_state {
    int n = 0;
    int dtype = 0;
    void *buf = nullptr;
    hipStream_t stream = nullptr;
    DeviceTables tables;
    void *d_red = nullptr;     // reduction partials and outputs
    size_t cap_red = 0;
    void *d_small = nullptr;   // constant coefficients (the X operator)
    size_t cap_small = 0;
    void *d_masks = nullptr;   // tables of qsim_expval
    size_t cap_masks = 0;
    void *h_table = nullptr;   // their pinned staging; draws and shots of qsim_sample
    size_t cap_table = 0;
    void *d_scan = nullptr;    // sampling: prefix sums
    size_t cap_scan = 0;
    double *h_out = nullptr;   // pinned readback, written by the reduction kernels
    size_t cap_out = 0;
    qsim_apply_stats last{};
};

struct qsim_program {
    int n = 0;
    int dtype = 0;
    Compiled c;
    DeviceTables dt;
    hipGraph_t graph = nullptr;
    hipGraphExec_t graph_exec = nullptr;
    void *graph_buf = nullptr;
    std::vector<hipEvent_t> events;
    size_t timed_passes = 0;
};

namespace {

// Device memory for reduction partials, and pinned memory (h->h_out) that the
// reductions write their results to.
int reduce_buffers(qsim_h h, size_t partial_doubles, size_t out_doubles, double **partials) {
    int rc = grow(&h->d_red, &h->cap_red, partial_doubles * sizeof(double), h->stream);
    if (rc) return rc;
    *partials = (double *)h->d_red;
    if (h->cap_out < out_doubles * sizeof(double)) {
        void *p = h->h_out;
        size_t cap = h->cap_out;
        rc = grow_host(&p, &cap, out_doubles * sizeof(double));
        if (rc) return rc;
        h->h_out = (double *)p;
        h->cap_out = cap;
    }
    return QSIM_OK;
}

// Two parts of a table into h->d_masks, through pinned memory: the copy is
// asynchronous and the call that makes it synchronises before it returns.
int upload_table(qsim_h h, const void *a, size_t na, const void *b, size_t nb) {
    int rc = grow(&h->d_masks, &h->cap_masks, na + nb, h->stream);
    if (!rc) rc = grow_host(&h->h_table, &h->cap_table, na + nb);
    if (rc) return rc;
    std::memcpy(h->h_table, a, na);
    if (nb) std::memcpy((char *)h->h_table + na, b, nb);
    return hip_rc(hipMemcpyAsync(h->d_masks, h->h_table, na + nb, hipMemcpyHostToDevice, h->stream));
}

// Marginal weights of qubits qs (unnormalised), into h->h_out[0 .. 2^nqs).
int marginal(qsim_h h, const int *qs, int nqs) {
    const uint32_t nch = qk::marginal_chunks(h->n, nqs);
    double *part;
    int rc = reduce_buffers(h, size_t(nch) << nqs, size_t(1) << nqs, &part);
    if (rc) return rc;
    // the sums go straight to the pinned read-back buffer
    rc = qk::launch_marginal(h->dtype, h->buf, 0, 1, h->n, qs, nqs, part, h->h_out, h->stream);
    if (rc) return rc;
    return hip_rc(hipStreamSynchronize(h->stream));
}

int weights01(qsim_h h, int q, double *P0, double *P1) {
    int rc = marginal(h, &q, 1);
    if (rc) return rc;
    *P0 = h->h_out[0];
    *P1 = h->h_out[1];
    return QSIM_OK;
}

}  // namespace

extern "C" {

int qsim_version(void) { return 1; }

int qsim_debug_fail_alloc(int after) {
    if (after < -1) return QSIM_E_ARG;
    qs::g_alloc_countdown.store(after);
    return QSIM_OK;
}

const char *qsim_last_error(void) { return g_last_error; }

const char *qsim_strerror(int s) {
    switch (s) {
    case QSIM_OK: return "ok";
    case QSIM_E_ARG: return "invalid argument";
    case QSIM_E_QUBIT: return "qubit out of range or repeated";
    case QSIM_E_NOMEM: return "out of memory";
    case QSIM_E_ZERO_PROB: return "asserted outcome has zero probability";
    case QSIM_E_NOT_DEFINITE: return "qubit is not in a definite state";
    case QSIM_E_HIP: return "HIP runtime error";
    case QSIM_E_CAPACITY: return "capacity exceeded";
    case QSIM_E_UNSUPPORTED: return "unsupported gate or option";
    default: return "unknown status";
    }
}

int qsim_create(int n, int dtype, void *dev_buf, size_t buf_bytes, void *hip_stream, qsim_h *out) {
    if (!out || n < 1 || n > kMaxQubits || (dtype != QSIM_C64 && dtype != QSIM_C128) || !dev_buf)
        return QSIM_E_ARG;
    if (buf_bytes < (size_t(1) << n) * elem_bytes(dtype)) return QSIM_E_CAPACITY;
    int rc = qk::init_kernels();
    if (rc) return rc;
    qsim_state *h = new (std::nothrow) qsim_state;
    if (!h) return QSIM_E_NOMEM;
    h->n = n;
    h->dtype = dtype;
    h->buf = dev_buf;
    h->stream = (hipStream_t)hip_stream;
    // constants: the X operator as one XOR-shift-1 diagonal (1, 1)
    rc = grow(&h->d_small, &h->cap_small, 4096, h->stream);
    if (rc) { delete h; return rc; }
    if (dtype == QSIM_C64) {
        float x[4] = {1, 0, 1, 0};
        rc = hip_rc(hipMemcpy(h->d_small, x, sizeof(x), hipMemcpyHostToDevice));
    } else {
        double x[4] = {1, 0, 1, 0};
        rc = hip_rc(hipMemcpy(h->d_small, x, sizeof(x), hipMemcpyHostToDevice));
    }
    if (!rc) rc = qk::launch_init_zero(dtype, dev_buf, 0, 1, n, h->stream);
    if (!rc) rc = hip_rc(hipStreamSynchronize(h->stream));
    if (rc) { qsim_destroy(h); return rc; }
    *out = h;
    return QSIM_OK;
}

int qsim_destroy(qsim_h h) {
    if (!h) return QSIM_E_ARG;
    (void)hipStreamSynchronize(h->stream);
    free_tables(&h->tables);
    if (h->d_red) (void)hipFree(h->d_red);
    if (h->d_small) (void)hipFree(h->d_small);
    if (h->d_masks) (void)hipFree(h->d_masks);
    if (h->d_scan) (void)hipFree(h->d_scan);
    if (h->h_out) (void)hipHostFree(h->h_out);
    if (h->h_table) (void)hipHostFree(h->h_table);
    delete h;
    return QSIM_OK;
}

int qsim_set_stream(qsim_h h, void *st) {
    if (!h) return QSIM_E_ARG;
    (void)hipStreamSynchronize(h->stream);
    h->stream = (hipStream_t)st;
    return QSIM_OK;
}

int qsim_stream_copy(void *dst, const void *src, size_t bytes, int flags, uint32_t rotate,
                     void *hip_stream) {
    if (!dst || !src || bytes % 16 || (flags & ~1)) return QSIM_E_ARG;
    return qk::launch_stream_copy(dst, src, bytes, (flags & 1) != 0, rotate, (hipStream_t)hip_stream);
}

int qsim_init_zero(qsim_h h) {
    if (!h) return QSIM_E_ARG;
    return qk::launch_init_zero(h->dtype, h->buf, 0, 1, h->n, h->stream);
}

int qsim_apply(qsim_h h, const qsim_gate *g, size_t ng, const double *mats, size_t n_mats,
               const double *params, size_t n_params, const qsim_fuse_opts *opt) {
    if (!h || (ng && !g)) return QSIM_E_ARG;
    TraceRange range("qsim_apply");
    Compiled c;
    int rc;
    try {
        rc = compile_circuit(h->n, h->dtype, g, ng, GateInputs{mats, n_mats, params, n_params}, opt, Spans::ONCE, &c);
    } catch (const std::bad_alloc &) {
        return QSIM_E_NOMEM;
    }
    if (rc) return rc;
    if (c.plan.ops.empty()) { h->last = c.stats; return QSIM_OK; }
    rc = upload_plan(&h->tables, h->dtype, c.plan, h->stream);
    if (rc) return rc;
    rc = enqueue_passes(c, h->tables, h->dtype, h->buf, h->stream, false);
    h->last = c.stats;
    return rc;
}

int qsim_compile(int n, int dtype, const qsim_gate *g, size_t ng, const double *mats,
                 size_t n_mats, const double *params, size_t n_params, const qsim_fuse_opts *opt,
                 qsim_prog *out) {
    if (!out || n < 1 || n > kMaxQubits || (dtype != QSIM_C64 && dtype != QSIM_C128) || (ng && !g))
        return QSIM_E_ARG;
    int rc = qk::init_kernels();
    if (rc) return rc;
    qsim_program *p = new (std::nothrow) qsim_program;
    if (!p) return QSIM_E_NOMEM;
    p->n = n;
    p->dtype = dtype;
    try {
        rc = compile_circuit(n, dtype, g, ng, GateInputs{mats, n_mats, params, n_params}, opt, Spans::REPLAY, &p->c);
    } catch (const std::bad_alloc &) {
        rc = QSIM_E_NOMEM;
    }
    if (!rc && !p->c.plan.ops.empty()) {
        rc = upload_plan(&p->dt, dtype, p->c.plan, nullptr);
        if (!rc) rc = hip_rc(hipStreamSynchronize(nullptr));
    }
    if (rc) { qsim_program_destroy(p); return rc; }
    *out = p;
    return QSIM_OK;
}

int qsim_run(qsim_h h, qsim_prog p) {
    if (!h || !p || h->n != p->n || h->dtype != p->dtype) return QSIM_E_ARG;
    TraceRange range("qsim_run");
    if (p->c.plan.ops.empty()) return QSIM_OK;
    if (p->graph_exec && p->graph_buf == h->buf) {
        return hip_rc(hipGraphLaunch(p->graph_exec, h->stream));
    }
    return enqueue_passes(p->c, p->dt, p->dtype, h->buf, h->stream, false);
}

int qsim_program_graph(qsim_prog p, qsim_h h, int enable) {
    if (!p || !h || h->n != p->n || h->dtype != p->dtype) return QSIM_E_ARG;
    if (p->graph_exec) { (void)hipGraphExecDestroy(p->graph_exec); p->graph_exec = nullptr; }
    if (p->graph) { (void)hipGraphDestroy(p->graph); p->graph = nullptr; }
    p->graph_buf = nullptr;
    if (!enable || p->c.plan.ops.empty()) return QSIM_OK;
    hipStream_t cs;
    if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) return QSIM_E_HIP;
    int rc = hip_rc(hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    if (!rc) {
        int erc = enqueue_passes(p->c, p->dt, p->dtype, h->buf, cs, false);
        hipGraph_t g = nullptr;
        rc = hip_rc(hipStreamEndCapture(cs, &g));
        if (!rc && erc) rc = erc;
        if (!rc) {
            p->graph = g;
            rc = hip_rc(hipGraphInstantiate(&p->graph_exec, g, nullptr, nullptr, 0));
        } else if (g) {
            (void)hipGraphDestroy(g);
        }
    }
    (void)hipStreamDestroy(cs);
    if (!rc) p->graph_buf = h->buf;
    return rc;
}

int qsim_run_timed(qsim_h h, qsim_prog p) {
    if (!h || !p || h->n != p->n || h->dtype != p->dtype) return QSIM_E_ARG;
    const size_t np = p->c.passes.size();
    if (p->events.size() < 2 * np) {
        for (size_t i = p->events.size(); i < 2 * np; i++) {
            hipEvent_t e;
            if (hipEventCreate(&e) != hipSuccess) return QSIM_E_HIP;
            p->events.push_back(e);
        }
    }
    for (size_t i = 0; i < np; i++) {
        if (hipEventRecord(p->events[2 * i], h->stream) != hipSuccess) return QSIM_E_HIP;
        const int rc = enqueue_pass(p->c, i, p->dt.d_ops, p->dt.d_coefs, 0, p->dtype, h->buf, 0, 1, nullptr, 0,
                                    h->stream);
        if (rc) return rc;
        if (hipEventRecord(p->events[2 * i + 1], h->stream) != hipSuccess) return QSIM_E_HIP;
    }
    p->timed_passes = np;
    return QSIM_OK;
}

int qsim_program_kernel_ms(qsim_prog p, double *ms, int64_t *launches) {
    if (!p || !ms || !launches) return QSIM_E_ARG;
    double tot = 0;
    for (size_t i = 0; i < p->timed_passes; i++) {
        if (hipEventSynchronize(p->events[2 * i + 1]) != hipSuccess) return QSIM_E_HIP;
        float f = 0;
        if (hipEventElapsedTime(&f, p->events[2 * i], p->events[2 * i + 1]) != hipSuccess) return QSIM_E_HIP;
        tot += f;
    }
    *ms = tot;
    *launches = int64_t(p->timed_passes);
    return QSIM_OK;
}

int qsim_program_stats(qsim_prog p, qsim_apply_stats *out) {
    if (!p || !out) return QSIM_E_ARG;
    *out = p->c.stats;
    return QSIM_OK;
}

int qsim_program_destroy(qsim_prog p) {
    if (!p) return QSIM_E_ARG;
    (void)hipDeviceSynchronize();
    if (p->graph_exec) (void)hipGraphExecDestroy(p->graph_exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    for (hipEvent_t e : p->events) (void)hipEventDestroy(e);
    free_tables(&p->dt);
    delete p;
    return QSIM_OK;
}

int qsim_last_stats(qsim_h h, qsim_apply_stats *out) {
    if (!h || !out) return QSIM_E_ARG;
    *out = h->last;
    return QSIM_OK;
}

int qsim_measure(qsim_h h, int q, double u, int *outcome, double *p_outcome) {
    if (!h || !outcome || !p_outcome) return QSIM_E_ARG;
    if (q < 0 || q >= h->n) return QSIM_E_QUBIT;
    if (!(u >= 0.0 && u < 1.0)) return QSIM_E_ARG;
    TraceRange range("qsim_measure");
    double P0, P1;
    int rc = weights01(h, q, &P0, &P1);
    if (rc) return rc;
    if (!(P0 + P1 > 0.0)) return QSIM_E_ZERO_PROB;
    const double p0 = P0 / (P0 + P1);
    const int o = (u < p0) ? 0 : 1;
    const double kept = o ? P1 : P0;
    rc = qk::launch_collapse(h->dtype, h->buf, h->n, q, o, 1.0 / std::sqrt(kept), h->stream);
    if (rc) return rc;
    *outcome = o;
    *p_outcome = kept / (P0 + P1);
    return QSIM_OK;
}

int qsim_measure_assert(qsim_h h, int q, int want, double *p_want) {
    if (!h || !p_want || (want != 0 && want != 1)) return QSIM_E_ARG;
    if (q < 0 || q >= h->n) return QSIM_E_QUBIT;
    TraceRange range("qsim_measure_assert");
    double P0, P1;
    int rc = weights01(h, q, &P0, &P1);
    if (rc) return rc;
    const double kept = want ? P1 : P0;
    if (!(kept > 0.0)) return QSIM_E_ZERO_PROB;
    rc = qk::launch_collapse(h->dtype, h->buf, h->n, q, want, 1.0 / std::sqrt(kept), h->stream);
    if (rc) return rc;
    *p_want = kept / (P0 + P1);
    return QSIM_OK;
}

int qsim_reset(qsim_h h, int q) {
    if (!h) return QSIM_E_ARG;
    if (q < 0 || q >= h->n) return QSIM_E_QUBIT;
    double P0, P1;
    int rc = weights01(h, q, &P0, &P1);
    if (rc) return rc;
    if (P1 == 0.0) return QSIM_OK;
    if (P0 != 0.0) return QSIM_E_NOT_DEFINITE;
    DevOp x{};
    x.coef = 0;
    x.present = 2u;   // shift 1: (X psi)[r] = psi[r ^ 1]
    x.k = 1;
    x.pos[0] = uint8_t(q);
    x.kind = DEVOP_MAT;
    return qk::launch_sweep(h->dtype, h->buf, 0, 1, h->n, x, h->d_small, h->stream);
}

int qsim_probs_noalloc(qsim_h h, const int *qs, int nqs, double *dev_out) {
    if (!h || !dev_out || nqs < 0 || nqs > 12 || (nqs && !qs)) return QSIM_E_ARG;
    int local[12];
    for (int i = 0; i < nqs; i++) {
        if (qs[i] < 0 || qs[i] >= h->n) return QSIM_E_QUBIT;
        for (int j = 0; j < i; j++)
            if (qs[j] == qs[i]) return QSIM_E_QUBIT;
        local[i] = qs[i];
    }
    return qk::launch_probs_noalloc(h->dtype, h->buf, h->n, local, nqs, dev_out, h->stream);
}

int qsim_norm(qsim_h h, double *out) {
    if (!h || !out) return QSIM_E_ARG;
    int rc = marginal(h, nullptr, 0);
    if (rc) return rc;
    *out = h->h_out[0];
    return QSIM_OK;
}

int qsim_probs(qsim_h h, const int *qs, int nqs, double *out) {
    if (!h || !out || nqs < 0 || nqs > 12 || (nqs && !qs)) return QSIM_E_ARG;
    for (int i = 0; i < nqs; i++) {
        if (qs[i] < 0 || qs[i] >= h->n) return QSIM_E_QUBIT;
        for (int j = 0; j < i; j++)
            if (qs[j] == qs[i]) return QSIM_E_QUBIT;
    }
    int rc = marginal(h, qs, nqs);
    if (rc) return rc;
    double tot = 0;
    for (int j = 0; j < (1 << nqs); j++) tot += h->h_out[j];
    if (!(tot > 0)) return QSIM_E_ZERO_PROB;
    for (int j = 0; j < (1 << nqs); j++) out[j] = h->h_out[j] / tot;
    return QSIM_OK;
}

int qsim_expval(qsim_h h, const qsim_pauli *t, size_t nt, double *out) {
    if (!h || !out || (nt && !t)) return QSIM_E_ARG;
    const uint64_t lim = (h->n >= 64) ? ~uint64_t(0) : ((uint64_t(1) << h->n) - 1);
    for (size_t k = 0; k < nt; k++) {
        if ((t[k].xmask & ~lim) || (t[k].zmask & ~lim) || !std::isfinite(t[k].coeff)) return QSIM_E_ARG;
    }
    TraceRange range("qsim_expval");
    if (nt == 0) {
        double nrm;
        const int rc = qsim_norm(h, &nrm);
        if (rc) return rc;
        if (!(nrm > 0)) return QSIM_E_ZERO_PROB;
        *out = 0.0;
        return QSIM_OK;
    }
    double nrm = 0.0, total = 0.0;
    int rc;
    try {
        ExpectPlan plan;
        if (plan_expect(h->n, h->dtype == QSIM_C64 ? 4 : 3, t, nt, &plan)) {
            // every term and the norm from one set of readings, one round trip
            const uint32_t nterms = uint32_t(nt) + 1;
            const uint32_t nch = qk::expect_chunks(h->n, plan.t, nterms, 1);
            double *part;
            rc = reduce_buffers(h, size_t(nch) * nterms, nterms, &part);
            if (!rc) rc = upload_table(h, plan.groups.data(), plan.groups.size() * sizeof(ExpectGroup),
                                       plan.recs.data(), plan.recs.size() * sizeof(DevOp));
            if (!rc) rc = qk::launch_expect(h->dtype, h->buf, 0, 1, h->n, plan, h->d_masks, nterms, nch, part,
                                            h->h_out, h->stream);
            const int src = hip_rc(hipStreamSynchronize(h->stream));
            if (rc || src) return rc ? rc : src;
            nrm = h->h_out[nt];
            if (!(nrm > 0)) return QSIM_E_ZERO_PROB;
            for (size_t k = 0; k < nt; k++) total += t[k].coeff * expect_value(t[k], h->h_out[k]);
            *out = total / nrm;
            return QSIM_OK;
        }
        rc = qsim_norm(h, &nrm);
        if (rc) return rc;
        if (!(nrm > 0)) return QSIM_E_ZERO_PROB;
        std::vector<uint64_t> table;
        const qk::PauliRows nrows = qk::pauli_rows(t, nt, &table);
        rc = upload_table(h, table.data(), 8 * table.size(), nullptr, 0);
        if (rc) return rc;
        const uint32_t nch = qk::pauli_chunks(h->n);
        double *part;
        rc = reduce_buffers(h, size_t(nch) * 2 * nt, 2 * nt, &part);
        if (rc) return rc;
        rc = qk::launch_pauli(h->dtype, h->buf, 0, 1, h->n, (const uint64_t *)h->d_masks, int(nt), nrows, part,
                              h->h_out, h->stream);
    } catch (const std::bad_alloc &) {
        return QSIM_E_NOMEM;
    }
    if (!rc) rc = hip_rc(hipStreamSynchronize(h->stream));
    if (rc) return rc;
    for (size_t k = 0; k < nt; k++) {
        const double re = h->h_out[2 * k], im = h->h_out[2 * k + 1];
        // <P> = Re(i^{#Y} S), S = sum_x (-1)^{popcount(x & z)} conj(a[x ^ x_mask]) a[x]
        double v;
        switch (__builtin_popcountll(t[k].xmask & t[k].zmask) & 3) {
        case 0: v = re; break;
        case 1: v = -im; break;
        case 2: v = -re; break;
        default: v = im; break;
        }
        total += t[k].coeff * v;
    }
    *out = total / nrm;
    return QSIM_OK;
}

int qsim_sample(qsim_h h, const double *u, size_t m, uint64_t *out) {
    if (!h || (m && (!u || !out))) return QSIM_E_ARG;
    for (size_t s = 0; s < m; s++)
        if (!(u[s] >= 0.0 && u[s] < 1.0)) return QSIM_E_ARG;
    TraceRange range("qsim_sample");
    // device scratch: seg | bsum[nb] | boff[nb + 1]; pinned: draws | shots, in
    // pieces of at most kPiece shots, read and written by the search itself
    const uint64_t nb = qk::scan_blocks(h->n), ns = qk::scan_segments(h->n);
    constexpr size_t kPiece = size_t(1) << 18;
    int rc = grow(&h->d_scan, &h->cap_scan, (ns + 2 * nb + 1) * 8, h->stream);
    double *part;
    if (!rc) rc = reduce_buffers(h, 0, 1, &part);
    if (!rc && m) rc = grow_host(&h->h_table, &h->cap_table, 16 * std::min(m, kPiece));
    if (rc) return rc;
    double *seg = (double *)h->d_scan, *bsum = seg + ns, *boff = bsum + nb;
    if ((rc = qk::launch_scan(h->dtype, h->buf, h->n, seg, bsum, boff, h->h_out, h->stream))) return rc;
    for (size_t at = 0; at < m || at == 0; at += kPiece) {
        const size_t k = std::min(m - at, kPiece);
        double *hu = (double *)h->h_table;
        uint64_t *hs = (uint64_t *)(hu + k);
        if (k) std::memcpy(hu, u + at, k * 8);
        if ((rc = qk::launch_search(h->dtype, h->buf, h->n, seg, boff, hu, k, hs, h->stream))) {
            (void)hipStreamSynchronize(h->stream);
            return rc;
        }
        if ((rc = hip_rc(hipStreamSynchronize(h->stream)))) return rc;
        if (at == 0 && !(h->h_out[0] > 0.0)) return QSIM_E_ZERO_PROB;
        if (k) std::memcpy(out + at, hs, k * 8);
    }
    return QSIM_OK;
}

int qsim_get_state(qsim_h h, void *dst) {
    if (!h || !dst) return QSIM_E_ARG;
    size_t bytes = (size_t(1) << h->n) * elem_bytes(h->dtype);
    if (hipMemcpyAsync(dst, h->buf, bytes, hipMemcpyDeviceToHost, h->stream) != hipSuccess) return QSIM_E_HIP;
    return hip_rc(hipStreamSynchronize(h->stream));
}

int qsim_set_state(qsim_h h, const void *src) {
    if (!h || !src) return QSIM_E_ARG;
    size_t bytes = (size_t(1) << h->n) * elem_bytes(h->dtype);
    if (hipMemcpyAsync(h->buf, src, bytes, hipMemcpyHostToDevice, h->stream) != hipSuccess) return QSIM_E_HIP;
    return hip_rc(hipStreamSynchronize(h->stream));
}

int qsim_autotune(qsim_h h, const qsim_gate *g, size_t ng, const double *mats, size_t n_mats,
                  const double *params, size_t n_params, size_t prefix_gates, qsim_fuse_opts *best,
                  double *ns_per_gate) {
    if (!h || !best || (ng && !g)) return QSIM_E_ARG;
    if (prefix_gates == 0) prefix_gates = 20000;
    // the prefix ends at a whole number of records; barriers are kept
    const size_t np = std::min(ng, prefix_gates);
    std::vector<qsim_fuse_opts> cands;
    const int tdef = (h->dtype == QSIM_C64 && h->n >= 23) ? 13 : 12;
    const int ldef = h->dtype == QSIM_C64 ? 4 : 3;
    const int wmax = h->dtype == QSIM_C64 ? 5 : 4;
    for (int t : {tdef - 1, tdef, tdef + 1}) {
        if (t > resident_max(h->dtype)) continue;
        for (int w = 2; w <= wmax; w++)
            for (float cost : {2.0f, 4.0f, 8.0f})
                for (int low : {ldef - 1, ldef}) {
                    qsim_fuse_opts o{};
                    o.level = 5;
                    o.max_width = w;
                    o.tile_qubits = t;
                    o.op_cost = cost;
                    o.low_qubits = low;
                    cands.push_back(o);
                }
    }
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return QSIM_E_HIP;
    double best_ns = 1e300;
    int rc = QSIM_OK, spans_tile = 0;
    uint64_t spans_low = 0;   // of the rotations timed on tiles of spans_tile qubits: a bit each
    DeviceTables dt;
    for (const qsim_fuse_opts &o : cands) {
        Compiled c;
        try {
            rc = compile_circuit(h->n, h->dtype, g, np, GateInputs{mats, n_mats, params, n_params}, &o, Spans::REPLAY, &c);
        } catch (const std::bad_alloc &) {
            rc = QSIM_E_NOMEM;
        }
        if (rc) break;
        if (c.plan.ops.empty()) continue;
        // fusion options do not change a plan of rotations: one candidate of each
        // tile (they follow each other) and number of low qubits
        if (o.tile_qubits != spans_tile) {
            spans_tile = o.tile_qubits;
            spans_low = 0;
        }
        if (c.pauli) {
            if ((spans_low >> o.low_qubits) & 1) continue;
            // (at the default width and cost, where every one gives it)
            if (c.fixed && (o.max_width != 4 || o.op_cost != 4.0f)) continue;
            spans_low |= uint64_t(1) << o.low_qubits;
        }
        if ((rc = upload_plan(&dt, h->dtype, c.plan, h->stream))) break;
        // warm, then time one run
        if ((rc = enqueue_passes(c, dt, h->dtype, h->buf, h->stream, false))) break;
        (void)hipEventRecord(e0, h->stream);
        if ((rc = enqueue_passes(c, dt, h->dtype, h->buf, h->stream, false))) break;
        (void)hipEventRecord(e1, h->stream);
        if ((rc = hip_rc(hipEventSynchronize(e1)))) break;
        float ms = 0;
        (void)hipEventElapsedTime(&ms, e0, e1);
        const double ns = 1e6 * double(ms) / double(std::max<int64_t>(1, c.stats.input_gates));
        if (ns < best_ns) {
            best_ns = ns;
            *best = o;
        }
    }
    free_tables(&dt);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (!rc) rc = qk::launch_init_zero(h->dtype, h->buf, 0, 1, h->n, h->stream);
    if (!rc) rc = hip_rc(hipStreamSynchronize(h->stream));
    if (ns_per_gate) *ns_per_gate = best_ns;
    return rc;
}

}  // extern "C"

namespace qs {

int tune_width(int n, int dtype, const qsim_gate *g, size_t ng, const GateInputs &in,
               const qsim_fuse_opts *base, Spans spans, int *best_w, double *best_ns) {
    const int wmax = dtype == QSIM_C64 ? 5 : 4;
    const size_t bytes = elem_bytes(dtype) << n;
    void *buf = nullptr;
    hipStream_t st = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int rc = hip_rc(hipMalloc(&buf, bytes));
    if (rc) return QSIM_E_NOMEM;
    if (!rc) rc = hip_rc(hipStreamCreate(&st));
    if (!rc) rc = hip_rc(hipEventCreate(&e0));
    if (!rc) rc = hip_rc(hipEventCreate(&e1));
    DeviceTables dt;
    *best_w = 0;
    *best_ns = 1e300;
    bool rotations = false;   // timed: the same plan at every width that takes it
    for (int w : {4, 2, 3, 5}) {
        if (w > wmax || rc) break;
        qsim_fuse_opts o{};
        if (base) o = *base;
        o.level = 5;
        o.max_width = w;
        Compiled c;
        try {
            rc = compile_circuit(n, dtype, g, ng, in, &o, spans, &c);
        } catch (const std::bad_alloc &) {
            rc = QSIM_E_NOMEM;
        }
        if (rc) break;
        if (c.plan.ops.empty()) {
            *best_w = w;
            *best_ns = 0.0;
            break;
        }
        if (c.pauli && rotations) continue;
        rotations = rotations || c.pauli;
        if ((rc = upload_plan(&dt, dtype, c.plan, st))) break;
        // warm, then the best of three timed runs
        if ((rc = enqueue_passes(c, dt, dtype, buf, st, true))) break;
        double best_run = 1e300;
        for (int rep = 0; rep < 3 && !rc; rep++) {
            (void)hipEventRecord(e0, st);
            if ((rc = enqueue_passes(c, dt, dtype, buf, st, true))) break;
            (void)hipEventRecord(e1, st);
            if ((rc = hip_rc(hipEventSynchronize(e1)))) break;
            float ms = 0;
            (void)hipEventElapsedTime(&ms, e0, e1);
            best_run = std::min(best_run, double(ms));
        }
        const double ns = 1e6 * best_run / double(std::max<int64_t>(1, c.stats.input_gates));
        if (!rc && ns < *best_ns) {
            *best_ns = ns;
            *best_w = w;
        }
        if (c.fixed) break;
    }
    if (st) (void)hipStreamSynchronize(st);
    free_tables(&dt);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (st) (void)hipStreamDestroy(st);
    (void)hipFree(buf);
    return rc;
}

int tune_tile_batch(int n, int dtype, const qsim_gate *g, size_t ng, const GateInputs &in,
                    const qsim_fuse_opts &base, Spans spans, uint32_t nstates, int *best_t) {
    *best_t = base.tile_qubits;
    if (n <= resident_max(dtype) || nstates == 0) return QSIM_OK;
    // enough states for 4,096 12-qubit tiles (16 per CU), within 1 GiB
    const size_t state_bytes = elem_bytes(dtype) << n;
    uint64_t sample = std::max<uint64_t>(1, uint64_t(4096) >> std::min(n - 12, 12));
    sample = std::min<uint64_t>(sample, nstates);
    sample = std::max<uint64_t>(1, std::min<uint64_t>(sample, (uint64_t(1) << 30) / state_bytes));
    void *buf = nullptr;
    hipStream_t st = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (alloc_fault() || hipMalloc(&buf, state_bytes * sample) != hipSuccess) {
        (void)hipGetLastError();
        return QSIM_E_NOMEM;
    }
    int rc = hip_rc(hipStreamCreate(&st));
    if (!rc) rc = hip_rc(hipEventCreate(&e0));
    if (!rc) rc = hip_rc(hipEventCreate(&e1));
    DeviceTables dt;
    double best_ms = 1e300;
    for (int t = 12; t <= 13 && !rc; t++) {
        qsim_fuse_opts o = base;
        o.tile_qubits = t;
        Compiled c;
        try {
            rc = compile_circuit(n, dtype, g, ng, in, &o, spans, &c);
        } catch (const std::bad_alloc &) {
            rc = QSIM_E_NOMEM;
        }
        if (rc) break;
        if (c.plan.ops.empty()) break;
        if ((rc = upload_plan(&dt, dtype, c.plan, st))) break;
        const uint64_t sstride = uint64_t(1) << n;
        // warm, then the best of three timed runs
        if ((rc = enqueue_passes(c, dt, dtype, buf, st, true, sstride, uint32_t(sample)))) break;
        double run_ms = 1e300;
        for (int rep = 0; rep < 3 && !rc; rep++) {
            (void)hipEventRecord(e0, st);
            if ((rc = enqueue_passes(c, dt, dtype, buf, st, true, sstride, uint32_t(sample)))) break;
            (void)hipEventRecord(e1, st);
            if ((rc = hip_rc(hipEventSynchronize(e1)))) break;
            float ms = 0;
            (void)hipEventElapsedTime(&ms, e0, e1);
            run_ms = std::min(run_ms, double(ms));
        }
        if (!rc && run_ms < best_ms) {
            best_ms = run_ms;
            *best_t = t;
        }
    }
    if (st) (void)hipStreamSynchronize(st);
    free_tables(&dt);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (st) (void)hipStreamDestroy(st);
    (void)hipFree(buf);
    return rc;
}

}  // namespace qs

extern "C" {

int qsim_debug_fuse(int n, const qsim_gate *g, size_t ng, const double *mats, size_t n_mats,
                    const double *params, size_t n_params, const qsim_fuse_opts *opt, int32_t *out_k, int32_t *out_qubits,
                    double *out_mats, size_t cap_ops, size_t cap_doubles, size_t *n_ops,
                    int64_t *counts) {
    if (n < 1 || n > kMaxQubits || (ng && !g) || !n_ops) return QSIM_E_ARG;
    FuseConfig fc;
    PlanConfig pc;
    default_configs(n, QSIM_C128, opt, &fc, &pc);
    if (opt && opt->max_width > 0) fc.max_width = std::max(1, std::min(opt->max_width, kMaxK));
    Lowered L;
    int rc;
    int64_t cnt[6];
    try {
        if (alloc_fault()) throw std::bad_alloc();
        rc = lower(n, g, ng, GateInputs{mats, n_mats, params, n_params}, false, false, &L);
        if (rc) return rc;
        fuse(n, &L, fc, cnt);
    } catch (const std::bad_alloc &) {
        return QSIM_E_NOMEM;
    }
    if (counts)
        for (int l = 0; l < 6; l++) counts[l] = cnt[l];
    *n_ops = L.ops.size();
    size_t need = 0;
    for (const Op &o : L.ops) need += 2 * size_t(o.dim()) * o.dim();
    if (L.ops.size() > cap_ops || need > cap_doubles) return QSIM_E_CAPACITY;
    size_t pos = 0;
    for (size_t i = 0; i < L.ops.size(); i++) {
        const Op &o = L.ops[i];
        out_k[i] = o.k;
        for (int j = 0; j < kMaxK; j++) out_qubits[5 * i + j] = j < o.k ? o.q[j] : -1;
        for (size_t e = 0; e < size_t(o.dim()) * o.dim(); e++) {
            out_mats[pos++] = o.m[e].real();
            out_mats[pos++] = o.m[e].imag();
        }
    }
    return QSIM_OK;
}

int qsim_parse_qasm(const char *text, size_t len, qsim_gate *out, size_t cap, size_t *n_out,
                    int32_t *n_qubits, int32_t *n_clbits) {
    if ((!text && len) || !n_out) return QSIM_E_ARG;
    std::vector<qsim_gate> g;
    int nq = 0, nc = 0;
    std::string err;
    int rc;
    try {
        rc = parse_qasm(text ? text : "", len, &g, &nq, &nc, &err);
    } catch (const std::bad_alloc &) {
        return QSIM_E_NOMEM;
    }
    if (rc) {
        std::snprintf(g_last_error, sizeof(g_last_error), "%s", err.c_str());
        return rc;
    }
    *n_out = g.size();
    if (n_qubits) *n_qubits = nq;
    if (n_clbits) *n_clbits = nc;
    if (g.size() > cap || (!out && !g.empty())) return QSIM_E_CAPACITY;
    if (!g.empty()) std::memcpy(out, g.data(), g.size() * sizeof(qsim_gate));
    return QSIM_OK;
}

int qsim_debug_plan(int n, int dtype, const qsim_gate *g, size_t ng, const double *mats,
                    size_t n_mats, const double *params, size_t n_params,
                    const qsim_fuse_opts *opt, qsim_apply_stats *out) {
    if (n < 1 || n > kMaxQubits || (dtype != QSIM_C64 && dtype != QSIM_C128) || !out) return QSIM_E_ARG;
    Compiled c;
    int rc;
    try {
        rc = compile_circuit(n, dtype, g, ng, GateInputs{mats, n_mats, params, n_params}, opt, Spans::ONCE, &c);
    } catch (const std::bad_alloc &) {
        return QSIM_E_NOMEM;
    }
    if (rc) return rc;
    *out = c.stats;
    return QSIM_OK;
}

}  // extern "C"
