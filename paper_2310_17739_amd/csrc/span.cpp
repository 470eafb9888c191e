// Pauli programs: circuits run as sequences of Pauli rotations.
//
// Lowering.  Most gates of the deep circuits of Section 5.1 are Clifford gates
// that cancel again: the basis changes and CNOT ladders around each Rz.  They
// are not applied to the state at all.  Going through the circuit, the state
// is psi = C phi with a Clifford frame C, and a rotation exp(-i phi P) on psi
// is the rotation exp(-i phi C^dagger P C) on phi, again a Pauli string (of
// any weight).  C is kept as the images C^dagger X_q C and C^dagger Z_q C of
// the generators.  Gates of the frame cancel structurally: a gate that undoes
// the last one on all of its wires removes it, so that what is left at the end
// of an epoch is an explicit gate list (empty for Pauli exponentials).  These
// gates run as operators of tiled passes after the epoch's rotations: an X or a
// CX moves amplitudes and leaves those that are 0 at 0, which rotations by a
// quarter turn would not.  A circuit with gates that are no product of few rotations
// (dense matrices, Toffolis) is not lowered this way.
//
// Passes.  A rotation mixes the amplitudes i and i ^ x only, x the string's X
// mask.  A pass therefore needs no tile of whole qubits: a tile is a coset of
// a t-dimensional subspace of GF(2)^n that holds the X masks of its rotations
// (and the low qubits, for contiguous chunks), so each rotation costs at most
// one dimension, whatever its weight, and its Z mask costs none: it is a sign,
// linear in the index.  Inside a pass, stages do the same for a thread's
// registers: with 2^r amplitudes per thread, a stage runs every rotation whose
// X mask is one of r independent ones, the bits of the register index, without
// any exchange, and only between stages the tile is re-laid out through LDS.
// (Sums of the r masks could run as well, but then the kernel has 2^r forms of
// a rotation in place of r, which outgrow the instruction cache.)  Rotations commute iff
// their strings do, so both levels may take a rotation past skipped ones that
// it commutes with.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>

#include "host.h"

namespace qs {

namespace {

// i^k times the Hermitian string i^|x & z| X^x Z^z
struct Pauli {
    uint64_t x = 0, z = 0;
    int k = 0;
};

Pauli mul(const Pauli &a, const Pauli &b) {
    Pauli r;
    r.x = a.x ^ b.x;
    r.z = a.z ^ b.z;
    r.k = (a.k + b.k + __builtin_popcountll(a.x & a.z) + __builtin_popcountll(b.x & b.z) +
           2 * __builtin_popcountll(a.z & b.x) - __builtin_popcountll(r.x & r.z)) & 3;
    return r;
}

bool anticommute(uint64_t ax, uint64_t az, uint64_t bx, uint64_t bz) {
    return __builtin_popcountll((ax & bz) ^ (az & bx)) & 1;
}
// The sign of -i (-i)^|x & z|, whose other part is 1 or i.
double kappa(uint64_t x, uint64_t z) { return (__builtin_popcountll(x & z) & 2) ? 1.0 : -1.0; }
// Whether exp(-i phi P) is a sign: phi a multiple of pi (sin phi <= least).
bool half_turns(double phi, double least = kTrivial) {
    const double a = std::fabs(phi);
    return a < 3.0 ? a <= least : std::fabs(std::sin(phi)) <= least;
}
// Whether a rotation does not commute with the string (x, z).
bool clash(const PauliOp &o, uint64_t x, uint64_t z) {
    return anticommute(x, z, o.x, o.z) || (o.two && anticommute(x, z, o.x, o.z2));
}

// The rotations of one epoch as a circuit is lowered.  Rotations about the same
// string add up past others that both commute with: what undoes each other leaves
// nothing, as products of matrices would, where one after the other they leave
// rounding errors.  Two strings of the same X mask whose angles cancel on half of
// the index space become one rotation of two angles.  It stays one, and only another
// about the same two strings adds to it, or a rotation that takes one of them
// away: half of it elsewhere would leave the other half's rounding errors where
// both are the identity.  (Phases of U1, T and CU1 add up all the same: a QFT has a
// rotation per controlled phase in place of two.)  `table` finds the latest rotation
// by X mask, a diagonal by its string; `prev` the one before.
class Rotations {
public:
    Rotations(PauliProgram *out, size_t most) : P(out), table(64) {
        dead.reserve(most);
        prev.reserve(most);
    }

    void add(PauliOp o, int epoch) {
        if (o.slot >= 0) return append(o, epoch);
        if (settle(&o)) return;
        int pair = -1;
        const int at = find(o.x, o.z, o.phi, o.phases, epoch, &pair);
        if (at >= 0) return merge(at, o.z, o.phi, o.phases);
        if (pair < 0) {
            if (second && spread(o, epoch)) return;
            return append(o, epoch);
        }
        PauliOp &c = P->ops[size_t(pair)];
        c.two = true;
        c.z2 = o.z;
        c.phi2 = o.phi;
        c.phases = c.phases && o.phases;
        changed = true;
        // (the pair may now undo an earlier one)
        const PauliOp t = c;
        const int same = find_pair(t, prev[size_t(pair)], pair);
        if (same < 0) return;
        dead[size_t(pair)] = 1;
        merge_pair(same, t);
    }
    // the commuting strings (x, z), (x, z2), as one
    void add_pair(PauliOp o, int epoch) {
        if (settle(&o)) return;
        if (!o.two) return add(o, epoch);
        const Entry &e = table[place(key(o.x, o.z), epoch)];
        const int same = e.epoch == epoch ? find_pair(o, e.head, int(P->ops.size())) : -1;
        if (same < 0) return append(o, epoch);
        merge_pair(same, o);
    }
    // Takes out what has cancelled, and gives half turns their exact form.  A half
    // turn is a string: it moves to the end of its epoch, where they are one, and
    // turns round the angles of those it does not commute with.  Then, and where
    // rotations have added up, others may meet that did not before.
    void finish() {
        bool again = changed;
        for (size_t i = 0; i < P->ops.size() && !again; i++) again = !dead[i] && half_turn(P->ops[i]);
        if (again) {
            std::vector<PauliOp> ops;
            std::vector<int> epochs;
            for (size_t i = 0; i < P->ops.size(); i++) {
                if (dead[i]) continue;
                ops.push_back(P->ops[i]);
                epochs.push_back(P->op_epoch[i]);
            }
            P->ops.clear();
            P->op_epoch.clear();
            dead.clear();
            prev.clear();
            table.assign(64, Entry{});
            used_epoch = -1;
            second = true;
            Pauli turns;   // the half turns so far, behind the rotations of their epoch
            for (size_t i = 0; i < ops.size(); i++) {
                PauliOp o = ops[i];
                if (anticommute(turns.x, turns.z, o.x, o.z)) {
                    if (o.slot < 0) o.phi = -o.phi;
                    else o.sign = -o.sign;
                }
                if (o.two && anticommute(turns.x, turns.z, o.x, o.z2)) o.phi2 = -o.phi2;
                if (half_turn(o)) turns = mul(turns, Pauli{o.x, o.z, std::sin(o.phi) > 0.0 ? 3 : 1});   // -i or i times it
                else if (o.two) add_pair(o, epochs[i]);
                else add(o, epochs[i]);
                if (i + 1 < ops.size() && epochs[i + 1] == epochs[i]) continue;
                P->phase += turns.k * (M_PI / 2);
                if (turns.x || turns.z) {
                    o = PauliOp{};
                    o.x = turns.x;
                    o.z = turns.z;
                    o.phi = M_PI / 2;
                    P->phase += M_PI / 2;
                    add(o, epochs[i]);
                }
                turns = Pauli{};
            }
        }
        size_t n = 0;
        for (size_t i = 0; i < P->ops.size(); i++) {
            if (dead[i]) continue;
            PauliOp &o = P->ops[i];
            if (o.x && half_turn(o)) {
                o.two = true;
                o.z2 = o.z;
                o.phi2 = 0.0;
            }
            if (n != i) {
                P->ops[n] = o;
                P->op_epoch[n] = P->op_epoch[i];
            }
            n++;
        }
        P->ops.resize(n);
        P->op_epoch.resize(n);
    }

private:
    PauliProgram *P;
    std::vector<char> dead;
    std::vector<int> prev;
    bool changed = false;   // a rotation has been added to another
    bool second = false;    // the rotations are gone through again
    struct Entry {
        uint64_t key = 0;
        int head = -1, epoch = -1;
    };
    std::vector<Entry> table;   // open addressing; entries of another epoch are free
    size_t used = 0;
    int used_epoch = -1;

    // (a half turn is at least pi/2 - 1e-14 away from 0)
    static bool half_turn(const PauliOp &o) {
        return o.slot < 0 && !o.two && std::fabs(o.phi) > 1.5 && std::fabs(std::cos(o.phi)) <= (o.x ? kTrivial : 1e-15);
    }
    static uint64_t key(uint64_t x, uint64_t z) { return x ? x : z | uint64_t(1) << 63; }
    size_t place(uint64_t k, int epoch) const {
        const size_t m = table.size() - 1;
        size_t i = size_t((k * 0x9e3779b97f4a7c15ull) >> 32) & m;
        while (table[i].epoch == epoch && table[i].key != k) i = (i + 1) & m;
        return i;
    }
    void append(const PauliOp &o, int epoch) {
        if (epoch != used_epoch) {
            used_epoch = epoch;
            used = 0;
        }
        if (2 * (used + 1) > table.size()) {
            std::vector<Entry> old(4 * table.size());
            old.swap(table);
            for (const Entry &e : old)
                if (e.epoch == epoch) table[place(e.key, epoch)] = e;
        }
        Entry &e = table[place(key(o.x, o.z), epoch)];
        const bool known = e.epoch == epoch;
        used += known ? 0 : 1;
        prev.push_back(known ? e.head : -1);
        e = Entry{key(o.x, o.z), int(P->ops.size()), epoch};
        dead.push_back(0);
        P->ops.push_back(o);
        P->op_epoch.push_back(epoch);
    }
    // Whether the rotations after c and before `from` commute with the string.
    bool reaches(int c, int from, uint64_t x, uint64_t z) const {
        for (int k = from - 1; k > c; k--)
            if (!dead[size_t(k)] && clash(P->ops[size_t(k)], x, z)) return false;
        return true;
    }
    // The rotation that one by phi about (x, z) adds to, if any; else *pair: one that
    // makes a rotation of two angles with it.  The search ends at a rotation that does
    // not commute with the string, and after kFar of those that do.
    int find(uint64_t x, uint64_t z, double phi, bool phase, int epoch, int *pair) const {
        const Entry &e = table[place(key(x, z), epoch)];
        if (e.epoch != epoch) return -1;
        int from = int(P->ops.size());
        for (int c = e.head; c >= 0 && int(P->ops.size()) - c <= kFar; c = prev[size_t(c)]) {
            if (!reaches(c, from, x, z)) return -1;
            from = c;
            if (dead[size_t(c)]) continue;
            const PauliOp &o = P->ops[size_t(c)];
            if (o.slot < 0 && (!o.two || (phase && o.phases)) && (o.z == z || (o.two && o.z2 == z))) return c;
            if (o.two && ((o.z == z && half_turns(o.phi + phi)) || (o.z2 == z && half_turns(o.phi2 + phi)))) return c;
            if (clash(o, x, z)) return -1;
            if (*pair < 0 && x && o.slot < 0 && !o.two) {
                const double a = kappa(x, o.z) * o.phi, b = kappa(x, z) * phi;
                if (half_turns(a + b) || half_turns(a - b)) *pair = c;
            }
        }
        return -1;
    }
    // The rotation of two angles about the strings of t before `from`, on the chain
    // from c, that t can be moved to.
    int find_pair(const PauliOp &t, int c, int from) const {
        for (; c >= 0 && int(P->ops.size()) - c <= kFar; c = prev[size_t(c)]) {
            if (!reaches(c, from, t.x, t.z) || !reaches(c, from, t.x, t.z2)) return -1;
            from = c;
            if (dead[size_t(c)]) continue;
            const PauliOp &o = P->ops[size_t(c)];
            if (o.two && ((o.z == t.z && o.z2 == t.z2) || (o.z == t.z2 && o.z2 == t.z))) return c;
            if (clash(o, t.x, t.z) || clash(o, t.x, t.z2)) return -1;
        }
        return -1;
    }
    // Several controlled rotations of one target, written with CX, may have been added
    // up: one string then has the angles of all others.  Takes that rotation and its
    // partners (o is the last of them) as rotations of two angles each, at the end.
    bool spread(const PauliOp &o, int epoch) {
        if (!o.x || o.phases) return false;
        const Entry &e = table[place(key(o.x, o.z), epoch)];
        if (e.epoch != epoch) return false;
        const int end = int(P->ops.size());
        std::vector<PauliOp> all{o};
        std::vector<int> at;
        for (int c = e.head; c >= 0 && end - c <= kFar && all.size() <= kSpread; c = prev[size_t(c)]) {
            const PauliOp &m = P->ops[size_t(c)];
            if (dead[size_t(c)] || m.slot >= 0 || m.two || m.phases) continue;
            bool free = reaches(c, end, m.x, m.z);
            for (const PauliOp &a : all) free = free && !clash(m, a.x, a.z);
            if (!free) break;
            all.push_back(m);
            at.push_back(c);
        }
        if (all.size() < 3) return false;
        // what the others take away from the largest, in the sign of either branch
        size_t h = 0;
        for (size_t j = 1; j < all.size(); j++)
            if (std::fabs(all[j].phi) > std::fabs(all[h].phi)) h = j;
        double rest = 0.0;
        for (size_t j = 0; j < all.size(); j++) rest += j == h ? 0.0 : kappa(all[j].x, all[j].z) * all[j].phi;
        const PauliOp hub = all[h];
        const double k = kappa(hub.x, hub.z), mine = k * hub.phi;
        const double sign = half_turns(mine + rest) ? -1.0 : 1.0;
        if (!half_turns(mine - sign * rest)) return false;
        P->phase += M_PI * std::nearbyint((mine - sign * rest) / M_PI);
        for (int c : at) dead[size_t(c)] = 1;
        for (size_t j = 0; j < all.size(); j++) {
            if (j == h) continue;
            PauliOp t = all[j];
            t.two = true;
            t.z2 = hub.z;
            t.phi2 = sign * k * kappa(t.x, t.z) * t.phi;
            append(t, epoch);
        }
        return true;
    }
    // Whether the rotation is none (a multiple of a half turn about its string: a
    // sign).  A diagonal leaves no amplitude out: it is none to the rounding of its
    // angle only.
    bool settle(PauliOp *o) {
        auto none = [&](double phi) {
            if (!half_turns(phi, o->x ? kTrivial : 5e-16)) return false;
            if (std::cos(phi) < 0.0) P->phase += M_PI;
            return true;
        };
        if (o->two && none(o->phi2)) o->two = false;
        if (!none(o->phi)) return false;
        if (!o->two) return true;
        o->z = o->z2;
        o->phi = o->phi2;
        o->two = false;
        return false;
    }
    void merge(int at, uint64_t z, double phi, bool phase) {
        PauliOp &c = P->ops[size_t(at)];
        c.phases = c.phases && phase;
        (c.z == z ? c.phi : c.phi2) += phi;
        settled(at);
    }
    void merge_pair(int at, const PauliOp &t) {
        PauliOp &c = P->ops[size_t(at)];
        c.phases = c.phases && t.phases;
        c.phi += c.z == t.z ? t.phi : t.phi2;
        c.phi2 += c.z == t.z ? t.phi2 : t.phi;
        settled(at);
    }
    // after the angles of rotation `at` have changed
    void settled(int at) {
        changed = true;
        if (settle(&P->ops[size_t(at)])) dead[size_t(at)] = 1;
        while (!dead.empty() && dead.back()) {
            const PauliOp &o = P->ops.back();
            table[place(key(o.x, o.z), P->op_epoch.back())].head = prev.back();
            P->ops.pop_back();
            P->op_epoch.pop_back();
            dead.pop_back();
            prev.pop_back();
        }
    }
    static constexpr int kFar = 4096;
    static constexpr size_t kSpread = 8;   // partners of one rotation
};

// A string on up to two qubits, as gates name it.
struct Axis {
    char l[2];
    int q[2];
    int k;
};

// The quarter turns of a rotation by theta: 1, 2 or 3 if theta is that many
// times pi/2 modulo 2 pi, to rounding, and 0 otherwise (whole turns included).
int quarter_turns(double theta) {
    const double t = theta / (M_PI / 2), r = std::nearbyint(t);
    if (std::fabs(r) > 3.0 || std::fabs(t - r) > 1e-15 * std::fabs(t)) return 0;
    return int(r) & 3;
}

struct Frame {
    struct Node {
        int kind, q0, q1;
        double theta;
        bool alive;
        int before[2];   // the live nodes before it on its wires
    };
    std::vector<Pauli> X, Z;
    std::vector<Node> nodes;
    std::vector<int> last;   // the last live node on each qubit's wire, or -1

    explicit Frame(int n) : X(size_t(n)), Z(size_t(n)), last(size_t(n)) { reset(); }
    void reset() {
        for (size_t q = 0; q < X.size(); q++) {
            X[q] = Pauli{uint64_t(1) << q, 0, 0};
            Z[q] = Pauli{0, uint64_t(1) << q, 0};
            last[q] = -1;
        }
        nodes.clear();
    }
    // C^dagger P C
    Pauli image(const Axis &a) const {
        Pauli r;
        for (int j = 0; j < a.k; j++) {
            const size_t q = size_t(a.q[j]);
            if (a.l[j] == 'X') r = mul(r, X[q]);
            else if (a.l[j] == 'Z') r = mul(r, Z[q]);
            else {
                r = mul(r, mul(X[q], Z[q]));
                r.k = (r.k + 1) & 3;   // Y = i X Z
            }
        }
        return r;
    }
    // images after a turn of `turns` quarters about the axis joins the frame
    void turn(const Axis &a, int turns) {
        const Pauli p = image(a);
        for (int j = 0; j < a.k; j++) {
            const size_t q = size_t(a.q[j]);
            for (int s = 0; s < 2; s++) {
                if ((a.l[j] == 'X' && s == 0) || (a.l[j] == 'Z' && s == 1)) continue;   // commutes
                Pauli &row = s == 0 ? X[q] : Z[q];
                if (turns == 2) row.k = (row.k + 2) & 3;
                else {
                    row = mul(row, p);
                    row.k = (row.k + (turns == 1 ? 3 : 1)) & 3;
                }
            }
        }
    }
    // Record a gate of the frame: it removes the last live node of all of its
    // wires if that is its inverse, else it becomes one.
    void push(int kind, int q0, int q1, double theta) {
        const int nq = q1 >= 0 ? 2 : 1;
        const int at = last[size_t(q0)];
        if (at >= 0 && (nq == 1 || last[size_t(q1)] == at)) {
            Node &h = nodes[size_t(at)];
            const bool same_q = (h.q0 == q0 && h.q1 == q1) ||
                                ((kind == QSIM_G_CZ || kind == QSIM_G_SWAP || kind == QSIM_G_RXX || kind == QSIM_G_RZZ) &&
                                 h.q0 == q1 && h.q1 == q0);
            bool inverse = same_q && h.kind == kind && h.theta == -theta;
            if (kind == QSIM_G_S || kind == QSIM_G_SDG)
                inverse = same_q && h.kind == (kind == QSIM_G_S ? QSIM_G_SDG : QSIM_G_S);
            if (kind == QSIM_G_SX) inverse = false;
            if (inverse) {
                h.alive = false;
                last[size_t(h.q0)] = h.before[0];
                if (nq == 2) last[size_t(h.q1)] = h.before[1];
                return;
            }
        }
        nodes.push_back({kind, q0, q1, theta, true, {at, nq == 2 ? last[size_t(q1)] : -1}});
        last[size_t(q0)] = int(nodes.size()) - 1;
        if (nq == 2) last[size_t(q1)] = int(nodes.size()) - 1;
    }
};

}  // namespace

uint64_t map_index(const IndexMap &m, uint64_t i) {
    if (m.z.empty()) return i;
    uint64_t r = 0;
    for (size_t q = 0; q < m.z.size(); q++) r |= uint64_t(__builtin_popcountll(i & m.z[q]) & 1) << q;
    return r;
}

bool pauli_lower(int n, const qsim_gate *g, const std::vector<size_t> &op_gate, const Lowered &L,
                 const GateInputs &in, bool keep_params, bool whole, PauliProgram *out) {
    const std::vector<int> &op_epoch = L.op_epoch;
    out->ops.clear();
    out->op_epoch.clear();
    out->recs.clear();
    out->left.clear();
    out->left_epoch.clear();
    out->map = IndexMap{};
    out->phase = 0.0;
    if (n > 48) return false;   // the device record keeps 48 bits of a Z mask
    Frame f(n);
    size_t extra = 0;
    int epoch = 0;
    out->ops.reserve(op_gate.size() / 4 + 16);
    // a rotation exp(-i phi P) about an axis seen through the frame
    Rotations rots(out, op_gate.size() / 4 + 16);
    size_t emitted = 0;
    auto emit = [&](const Pauli &p, double phi, int slot, bool phases = false) {
        PauliOp o;
        o.phases = phases;
        o.x = p.x;
        o.z = p.z;
        o.slot = slot;
        const double sign = (p.k & 2) ? -1.0 : 1.0;
        if (slot < 0) o.phi = sign * phi;
        else o.sign = sign;
        rots.add(o, epoch);
        emitted++;
    };
    // rotations about two axes of commuting strings, as one where their X masks agree
    auto emit_pair = [&](const Pauli &p, double phi, const Pauli &p2, double phi2) {
        if (p.x != p2.x || !p.x) {
            emit(p, phi, -1);
            emit(p2, phi2, -1);
            return;
        }
        PauliOp o;
        o.x = p.x;
        o.z = p.z;
        o.phi = (p.k & 2) ? -phi : phi;
        o.two = true;
        o.z2 = p2.z;
        o.phi2 = (p2.k & 2) ? -phi2 : phi2;
        rots.add_pair(o, epoch);
        emitted += 2;
    };
    auto one = [](char l, int q) { return Axis{{l, 'I'}, {q, -1}, 1}; };
    auto two = [](char a, int qa, char b, int qb) { return Axis{{a, b}, {qa, qb}, 2}; };
    // the live gates of the frame, to run after the epoch's rotations
    auto flush = [&]() {
        for (const Frame::Node &h : f.nodes) {
            if (!h.alive) continue;
            qsim_gate r{};
            r.kind = uint16_t(h.kind);
            r.nq = h.q1 >= 0 ? 2 : 1;
            r.q[0] = h.q0;
            r.q[1] = std::max(h.q1, 0);
            r.slot = -1;
            r.theta[0] = h.theta;
            out->left.push_back(r);
            out->left_epoch.push_back(epoch);
            // what it would take as rotations
            extra += h.kind == QSIM_G_SWAP ? 9 : h.kind == QSIM_G_H || h.kind == QSIM_G_CX || h.kind == QSIM_G_CY ||
                     h.kind == QSIM_G_CZ ? 3 : 1;
        }
        f.reset();
    };
    // the frame as a map of the basis states; false if it is none
    auto as_map = [&](IndexMap *m) {
        m->z.resize(size_t(n));
        m->c = 0;
        bool same = true;
        for (int q = 0; q < n; q++) {
            const Pauli &z = f.Z[size_t(q)];
            if (z.x) return false;
            m->z[size_t(q)] = z.z;
            if (z.k) m->c |= uint64_t(1) << q;
            same = same && z.z == (uint64_t(1) << q);
        }
        if (same && !m->c) m->z.clear();
        return true;
    };
    // the records before epoch e, seen through the frame
    size_t next_rec = 0;
    auto records = [&](int e) {
        for (; next_rec < L.meas.size() && L.meas[next_rec].epoch < e; next_rec++) {
            PauliRecord r;
            r.rec = L.meas[next_rec];
            const Pauli &z = f.Z[size_t(r.rec.q)], &x = f.X[size_t(r.rec.q)];
            if (z.x) return false;
            r.z = z.z;
            r.flip = z.k != 0;
            if (r.rec.kind == DEVOP_RESET || r.rec.kind == DEVOP_MEASURE_RESET) {
                if (x.z || x.k) return false;
                r.x = x.x;
            }
            // (gates that are diagonal leave phases behind a map of indices)
            for (const Frame::Node &h : f.nodes)
                if (h.alive && h.kind != QSIM_G_CX && h.kind != QSIM_G_SWAP && h.kind != QSIM_G_X) return false;
            if (!as_map(&r.map)) return false;
            out->recs.push_back(std::move(r));
        }
        return true;
    };
    for (size_t j = 0; j < op_gate.size(); j++) {
        const qsim_gate &gi = g[op_gate[j]];
        if (op_epoch[j] != epoch) {
            if (!whole) flush();
            else if (!records(op_epoch[j])) return false;
            epoch = op_epoch[j];
        }
        // records that the matrix lowering refuses are left to it
        const int k = gi.nq;
        const int kind = gi.kind;
        const bool wide = kind >= QSIM_G_CX && kind <= QSIM_G_RZZ;
        if (k != (wide ? 2 : 1) || (!wide && (kind > QSIM_G_U3 || kind < QSIM_G_ID))) return false;
        const int q0 = gi.q[0], q1 = wide ? gi.q[1] : -1;
        if (q0 < 0 || q0 >= n || (wide && (q1 < 0 || q1 >= n || q1 == q0))) return false;
        for (double v : gi.theta)
            if (!std::isfinite(v)) return false;
        double th = gi.theta[0];
        const bool linear = kind == QSIM_G_RX || kind == QSIM_G_RY || kind == QSIM_G_RZ || kind == QSIM_G_RXX ||
                            kind == QSIM_G_RZZ;
        int slot = -1;
        if (gi.slot >= 0) {
            if (size_t(gi.slot) >= in.n_params) return false;
            if (keep_params) {
                if (!linear) return false;
                slot = gi.slot;
            } else {
                if (!in.params || !std::isfinite(in.params[gi.slot])) return false;
                th = in.params[gi.slot];
            }
        }
        auto rotation = [&](const Axis &a, double theta) {
            const int turns = slot < 0 ? quarter_turns(theta) : 0;
            if (turns) {
                f.turn(a, turns);
                f.push(kind, q0, q1, theta);
            } else {
                emit(f.image(a), theta / 2, slot);
            }
        };
        switch (kind) {
        case QSIM_G_ID: break;
        case QSIM_G_H:
            std::swap(f.X[size_t(q0)], f.Z[size_t(q0)]);
            f.push(kind, q0, -1, 0.0);
            break;
        case QSIM_G_X: f.turn(one('X', q0), 2); f.push(kind, q0, -1, 0.0); break;
        case QSIM_G_Y: f.turn(one('Y', q0), 2); f.push(kind, q0, -1, 0.0); break;
        case QSIM_G_Z: f.turn(one('Z', q0), 2); f.push(kind, q0, -1, 0.0); break;
        case QSIM_G_S: f.turn(one('Z', q0), 1); f.push(kind, q0, -1, 0.0); break;
        case QSIM_G_SDG: f.turn(one('Z', q0), 3); f.push(kind, q0, -1, 0.0); break;
        case QSIM_G_SX: f.turn(one('X', q0), 1); f.push(kind, q0, -1, 0.0); break;
        case QSIM_G_T: emit(f.image(one('Z', q0)), M_PI / 8, -1, true); out->phase += M_PI / 8; break;
        case QSIM_G_TDG: emit(f.image(one('Z', q0)), -M_PI / 8, -1, true); out->phase -= M_PI / 8; break;
        case QSIM_G_RX: rotation(one('X', q0), th); break;
        case QSIM_G_RY: rotation(one('Y', q0), th); break;
        case QSIM_G_RZ: rotation(one('Z', q0), th); break;
        case QSIM_G_RXX: rotation(two('X', q0, 'X', q1), th); break;
        case QSIM_G_RZZ: rotation(two('Z', q0, 'Z', q1), th); break;
        case QSIM_G_U1: emit(f.image(one('Z', q0)), th / 2, -1, true); out->phase += th / 2; break;
        case QSIM_G_U2:
        case QSIM_G_U3: {
            // e^{i (ph + la) / 2} Rz(ph) Ry(t) Rz(la)
            const double t = kind == QSIM_G_U2 ? M_PI / 2 : th;
            const double ph = kind == QSIM_G_U2 ? th : gi.theta[1];
            const double la = kind == QSIM_G_U2 ? gi.theta[1] : gi.theta[2];
            emit(f.image(one('Z', q0)), la / 2, -1);
            emit(f.image(one('Y', q0)), t / 2, -1);
            emit(f.image(one('Z', q0)), ph / 2, -1);
            out->phase += (ph + la) / 2;
            break;
        }
        case QSIM_G_CX: {
            Pauli &xc = f.X[size_t(q0)], &zt = f.Z[size_t(q1)];
            xc = mul(xc, f.X[size_t(q1)]);
            zt = mul(f.Z[size_t(q0)], zt);
            f.push(kind, q0, q1, 0.0);
            break;
        }
        case QSIM_G_CY: {
            const Pauli y = f.image(one('Y', q1));
            f.X[size_t(q0)] = mul(f.X[size_t(q0)], y);
            f.X[size_t(q1)] = mul(f.Z[size_t(q0)], f.X[size_t(q1)]);
            f.Z[size_t(q1)] = mul(f.Z[size_t(q0)], f.Z[size_t(q1)]);
            f.push(kind, q0, q1, 0.0);
            break;
        }
        case QSIM_G_CZ: {
            const Pauli zc = f.Z[size_t(q0)], zt = f.Z[size_t(q1)];
            f.X[size_t(q0)] = mul(f.X[size_t(q0)], zt);
            f.X[size_t(q1)] = mul(f.X[size_t(q1)], zc);
            f.push(kind, q0, q1, 0.0);
            break;
        }
        case QSIM_G_SWAP:
            std::swap(f.X[size_t(q0)], f.X[size_t(q1)]);
            std::swap(f.Z[size_t(q0)], f.Z[size_t(q1)]);
            f.push(kind, q0, q1, 0.0);
            break;
        case QSIM_G_CRX:
        case QSIM_G_CRY:
        case QSIM_G_CRZ: {
            // exp(-i theta/2 (1 - Z_c)/2 P)
            const char l = kind == QSIM_G_CRX ? 'X' : kind == QSIM_G_CRY ? 'Y' : 'Z';
            emit_pair(f.image(one(l, q1)), th / 4, f.image(two('Z', q0, l, q1)), -th / 4);
            break;
        }
        case QSIM_G_CU1:
            // exp(i theta (1 - Z_c)(1 - Z_t) / 4)
            emit(f.image(one('Z', q0)), th / 4, -1, true);
            emit(f.image(one('Z', q1)), th / 4, -1, true);
            emit(f.image(two('Z', q0, 'Z', q1)), -th / 4, -1, true);
            out->phase += th / 4;
            break;
        default: return false;   // CH, CU3: no product of few rotations
        }
    }
    if (whole) {
        if (!records(L.n_epochs)) return false;
        bool permutes = true;
        for (const Frame::Node &h : f.nodes)
            permutes = permutes && (!h.alive || h.kind == QSIM_G_CX || h.kind == QSIM_G_SWAP || h.kind == QSIM_G_X);
        if (permutes && as_map(&out->map)) f.reset();
        else epoch = L.n_epochs;   // what is left follows every record
    }
    flush();
    rots.finish();
    // With many gates left in the frame, the fused operators of the matrix lowering
    // do less.  Span passes against tiled ones, us, random rotations and Clifford
    // gates with so many left per rotation: 21 qubits complex128 0.1 162 (170), 0.3
    // 170 (162), 1.6 191 (172), 24 qubits complex64 0.3 630 (603), 1.1 588 (571), 3.2
    // 674 (527); layers of RY, RZ and CX, 1.4 left, 634 (363) and 2321 (1494).
    return 3 * extra <= emitted;
}

// -------------------------------------------------------------- planning
namespace {

// A subspace of GF(2)^n in reduced echelon form: vector v[j] is the only one
// with bit piv[j].
struct Span {
    uint64_t v[16];
    int piv[16];
    int d = 0;
    uint64_t pm = 0;                 // pivot bits
    int8_t at[64];                   // vector of each pivot bit

    uint64_t reduce(uint64_t x) const {
        for (uint64_t m = x & pm; m; m &= m - 1) x ^= v[at[__builtin_ctzll(m)]];
        return x;
    }
    // adds x, already reduced and not 0
    void add(uint64_t x) {
        const int p = 63 - __builtin_clzll(x);
        for (int j = 0; j < d; j++)
            if ((v[j] >> p) & 1) v[j] ^= x;
        v[d] = x;
        piv[d] = p;
        at[p] = int8_t(d);
        pm |= uint64_t(1) << p;
        d++;
    }
    // the coordinates of a member: its pivot bits
    uint32_t coords(uint64_t x) const {
        uint32_t c = 0;
        for (int j = 0; j < d; j++) c |= uint32_t((x >> piv[j]) & 1) << j;
        return c;
    }
};

// The same for small masks, for tests of independence only.
struct Rank {
    uint32_t v[32];
    uint32_t have = 0;
    // x without what was added: 0 if it depends on that
    uint32_t rest(uint32_t x) const {
        while (x) {
            const int p = 31 - __builtin_clz(x);
            if (!((have >> p) & 1)) break;
            x ^= v[p];
        }
        return x;
    }
    // adds a rest that is not 0
    void put(uint32_t r) {
        const int p = 31 - __builtin_clz(r);
        v[p] = r;
        have |= 1u << p;
    }
    // whether x is independent of what was added (and adds it)
    bool add(uint32_t x) {
        const uint32_t r = rest(x);
        if (r) put(r);
        return r != 0;
    }
};

// LDS slot of tile coordinates c: the coordinates from 5 up are folded into
// the low 5 bits (the banks: 32 elements of 8 bytes or 16 of 16), so that a
// layout finds lanes on distinct banks whichever coordinates its registers
// take.  Linear and a bijection.
constexpr uint32_t kBank[9] = {1, 2, 4, 8, 19, 22, 5, 10, 31};
uint32_t span_slot(uint32_t c) {
    uint32_t s = c;
    for (int j = 5; j < 14; j++)
        if ((c >> j) & 1) s ^= kBank[j - 5];
    return s;
}

// Rotations skipped by one pass (or stage) after which it is closed: a later one has to
// commute with all of them, and a longer list finds hardly any on the
// benchmark circuits.
constexpr size_t kSkipMax = 64;
// Rotations of one pass.
constexpr size_t kPassMax = 96;
// Bits that the rotations whose angle is known here may grow a state by before
// the scale is applied, for double and single precision.  Those bound per state
// grow it by half a bit each at most, kPassMax / 2 in a pass, and one rotation
// beyond the limit by 1 / kLeastCos: 20 + 48 + 53 of the 127 bits of a float.
constexpr double kGrownMost[2] = {400.0, 20.0};

// The layout of a stage whose registers run the directions `dirs` (at most
// `regs` independent vectors of T), as tile coordinates.
void stage_layout(const Span &T, const std::vector<uint64_t> &dirs, int t, int c, int regs, SpanStage *st) {
    const int logt = t - regs;
    uint32_t reg[8];
    int nr = 0;
    Rank all;
    for (uint64_t x : dirs) {
        reg[nr] = T.coords(x);
        all.add(reg[nr++]);
    }
    // spare register bits: the highest coordinates that are free
    for (int j = t - 1; j >= 0 && nr < regs; j--)
        if (all.add(1u << j)) reg[nr++] = 1u << j;
    // lanes: the low qubits first (contiguous chunks in memory), then
    // coordinates that bring the lanes of an LDS access to distinct banks,
    // then the others
    int nt = 0;
    uint32_t thr[16], taken = 0;
    Rank bank;
    auto take = [&](int j) {
        thr[nt++] = 1u << j;
        taken |= 1u << j;
    };
    for (int j = 0; j < c && nt < logt; j++) {
        if (!all.add(1u << j)) continue;
        bank.add(span_slot(1u << j) & 31u);
        take(j);
    }
    for (int j = c; j < t && nt < std::min(5, logt); j++) {
        if ((taken >> j) & 1) continue;
        const uint32_t r = all.rest(1u << j), rb = bank.rest(span_slot(1u << j) & 31u);
        if (!r || !rb) continue;
        all.put(r);
        bank.put(rb);
        take(j);
    }
    for (int j = 0; j < t && nt < logt; j++)
        if (!((taken >> j) & 1) && all.add(1u << j)) take(j);
    for (int j = 0; j < logt; j++) st->layout[j] = uint16_t(thr[j]);
    for (int j = 0; j < regs; j++) st->layout[logt + j] = uint16_t(reg[j]);
}

// Stages for the items of a pass (rotations i of P, and ~i for its records) in
// their order: each takes what its registers can run, rotations past skipped
// ones that they commute with, and ends at a record that it cannot take.
void make_stages(const PauliProgram &P, const std::vector<int> &items, const Span &T, int t, int c, int regs,
                 std::vector<SpanStage> *stages) {
    struct Mask {
        uint64_t x, z;
    };
    std::vector<Mask> skipped;
    std::vector<int> left = items, later;
    while (!left.empty()) {
        Span R;
        SpanStage st;
        std::vector<uint64_t> dirs;   // the masks that are register bits
        skipped.clear();
        later.clear();
        bool closed = false;
        auto fits = [&](uint64_t x) {
            if (!x || std::find(dirs.begin(), dirs.end(), x) != dirs.end()) return true;
            const uint64_t r = R.reduce(x);
            if (!r || R.d >= regs) return false;
            R.add(r);
            dirs.push_back(x);
            return true;
        };
        for (int i : left) {
            if (closed || skipped.size() >= kSkipMax) {
                later.push_back(i);
                continue;
            }
            if (i < 0) {
                // nothing passes a record
                if (later.empty() && fits(P.recs[size_t(~i)].x)) {
                    st.ops.push_back(i);
                } else {
                    later.push_back(i);
                    closed = true;
                }
                continue;
            }
            const PauliOp &o = P.ops[size_t(i)];
            bool free = true;
            for (const Mask &s : skipped)
                if (clash(o, s.x, s.z)) {
                    free = false;
                    break;
                }
            if (free && fits(o.x)) {
                st.ops.push_back(i);
            } else {
                skipped.push_back({o.x, o.z});
                if (o.two) skipped.push_back({o.x, o.z2});
                later.push_back(i);
            }
        }
        left.swap(later);
        stage_layout(T, dirs, t, c, regs, &st);
        stages->push_back(std::move(st));
    }
}

// A stage record: the LDS slots of the layout's positions.
DevOp stage_record(const SpanStage &st, int t, int number) {
    DevOp h{};
    h.kind = DEVOP_STAGE;
    h.kx = uint8_t(number);
    uint8_t *raw = reinterpret_cast<uint8_t *>(&h);
    for (int j = 0; j < t; j++) {
        const uint16_t s = uint16_t(span_slot(st.layout[j]));
        std::memcpy(raw + (j < 7 ? 2 * j : 16 + 2 * (j - 7)), &s, 2);
    }
    return h;
}

// The form and the sign masks of the string (x, z) in a layout whose positions
// move the state's index by V; false if x is none of its register bits.
bool string_record(uint64_t x, uint64_t z, const uint64_t *V, int t, int regs, DevOp *d) {
    const int logt = t - regs;
    int bit = -1;
    for (int r = 0; r < regs; r++)
        if (V[logt + r] == x) bit = r;
    if (x && bit < 0) return false;
    d->k = uint8_t(x ? 2 * bit + (__builtin_popcountll(x & z) & 1) : 2 * regs);
    uint32_t zr = 0, zt = 0;
    for (int b = 0; b < regs; b++) zr |= uint32_t(__builtin_popcountll(z & V[logt + b]) & 1) << b;
    for (int b = 0; b < logt; b++) zt |= uint32_t(__builtin_popcountll(z & V[b]) & 1) << b;
    d->present = zr;
    d->slot[0] = uint16_t(zt);
    for (int b = 0; b < 3; b++) d->slot[1 + b] = uint16_t((z >> (16 * b)) & 0xffff);
    return true;
}

}  // namespace

void plan_spans(int n, const PauliProgram &P, int t, int c, int regs, size_t meta_budget, int window,
                bool full, int first, int last, std::vector<Pass> *passes) {
    const size_t N = size_t(last - first);
    std::vector<int> nxt(N + 1), prv(N + 1);
    const int head = int(N);
    for (size_t i = 0; i <= N; i++) {
        nxt[i] = i < N ? int(i) + 1 : 0;
        prv[i] = i > 0 ? int(i) - 1 : int(N);
    }
    if (N == 0) return;
    const PauliOp *ops = P.ops.data() + first;
    struct Mask {
        uint64_t x, z;
    };
    std::vector<Mask> skipped;
    skipped.reserve(kSkipMax + 2);
    // may o run before every skipped rotation?
    auto passes_by = [&](const PauliOp &o) {
        for (const Mask &s : skipped)
            if (clash(o, s.x, s.z)) return false;
        return true;
    };
    while (nxt[size_t(head)] != head) {
        Span T;
        for (int q = 0; q < c; q++) T.add(uint64_t(1) << q);
        // the space with o in it; false if it grows beyond t dimensions
        auto grow = [&](const PauliOp &o) {
            if (!full) {
                const uint64_t r = T.reduce(o.x);
                if (r && T.d >= t) return false;
                if (r) T.add(r);
                return true;
            }
            Span U = T;
            for (uint64_t m = o.x | o.z | o.z2; m; m &= m - 1) {
                const uint64_t r = U.reduce(m & (~m + 1));
                if (r && U.d >= t) return false;
                if (r) U.add(r);
            }
            T = U;
            return true;
        };
        std::vector<int> sel;
        skipped.clear();
        size_t meta = 0;
        int scanned = 0;
        for (int i = nxt[size_t(head)]; i != head && scanned < window && skipped.size() < kSkipMax && sel.size() < kPassMax;
             i = nxt[size_t(i)], scanned++) {
            const PauliOp &o = ops[i];
            // LDS of its entries and factors; it may open a stage of its own
            const size_t need = 24 * size_t(o.entries()) + 88;
            if ((sel.empty() || meta + need <= meta_budget) && passes_by(o) && grow(o)) {
                sel.push_back(i);
                meta += need;
            } else {
                skipped.push_back({o.x, o.z});
                if (o.two) skipped.push_back({o.x, o.z2});
            }
        }
        for (int i : sel) {
            nxt[size_t(prv[size_t(i)])] = nxt[size_t(i)];
            prv[size_t(nxt[size_t(i)])] = prv[size_t(i)];
        }
        for (int q = 0; q < n && T.d < t; q++) {
            const uint64_t r = T.reduce(uint64_t(1) << q);
            if (r) T.add(r);
        }
        Pass p;
        p.kind = Pass::TILE;
        p.t = t;
        p.c = c;
        p.span = true;
        p.tile_mask = T.pm;
        for (int &i : sel) i += first;
        make_stages(P, sel, T, t, c, regs, &p.stages);
        for (int j = 0; j < t; j++) p.span_v[j] = T.v[j];
        passes->push_back(std::move(p));
    }
}

void plan_whole(int n, const PauliProgram &P, int n_epochs, int c, int regs, size_t meta_budget,
                std::vector<Pass> *passes) {
    Span T;
    for (int q = 0; q < n; q++) T.add(uint64_t(1) << q);
    std::vector<int> items;
    size_t meta = 0;
    auto close = [&]() {
        if (items.empty()) return;
        Pass p;
        p.kind = Pass::TILE;
        p.t = n;
        p.c = std::min(c, n);
        p.span = true;
        p.tile_mask = T.pm;
        make_stages(P, items, T, n, p.c, regs, &p.stages);
        for (int j = 0; j < n; j++) p.span_v[j] = T.v[j];
        passes->push_back(std::move(p));
        items.clear();
        meta = 0;
    };
    auto take = [&](int i, size_t bytes) {
        if (!items.empty() && (meta + bytes > meta_budget || items.size() >= kPassMax)) close();
        items.push_back(i);
        meta += bytes;
    };
    size_t at = 0, r = 0;
    for (int e = 0; e <= n_epochs; e++) {
        // LDS of entries, factors and a stage of its own; a record's layout
        for (; at < P.ops.size() && P.op_epoch[at] == e; at++) take(int(at), 24 * size_t(P.ops[at].entries()) + 88);
        for (; r < P.recs.size() && P.recs[r].rec.epoch == e; r++) take(~int(r), 24 + 88 + 88);
    }
    close();
}

uint64_t span_vector(const Pass &p, uint32_t coords) {
    uint64_t x = 0;
    for (; coords; coords &= coords - 1) x ^= p.span_v[__builtin_ctz(coords)];
    return x;
}

int pack_span_pass(const PauliProgram &P, const Pass &p, int regs, bool single, PackedPlan *out, uint32_t *run) {
    const int t = p.t;
    std::vector<DevOp> behind;   // the layouts that failing records store in
    double grown = 0.0;   // bits that the state may have grown by since the scale was last applied
    const size_t before = out->ops.size();
    auto dummy = [&]() {
        out->op_np.push_back(0);
        for (int j = 0; j < 3; j++) out->op_slots.push_back(-1);
        for (int j = 0; j < 2; j++) out->coefs.push_back(cd(0.0, 0.0));
    };
    int number = 0;
    for (const SpanStage &st : p.stages) {
        out->ops.push_back(stage_record(st, t, number++));
        dummy();   // (the kernel reads two coefficients of every record)
        // the layout's positions as vectors of the state's index
        uint64_t V[16];
        for (int j = 0; j < t; j++) V[j] = span_vector(p, st.layout[j]);
        for (int idx : st.ops) {
            if (idx < 0) {
                const PauliRecord &r = P.recs[size_t(~idx)];
                DevOp d{};
                if (!string_record(r.x, r.z, V, t, regs, &d)) return QSIM_E_ARG;
                d.kind = DEVOP_SPAN_REC;
                d.pos[0] = uint8_t(r.rec.kind);
                d.present |= (r.x ? uint32_t(d.k / 2 + 1) : 0u) << 4 | uint32_t(r.flip) << 7;
                for (int b = 1; b < 5; b++) d.slot[b] = 0;
                d.slot[1] = uint16_t(uint32_t(r.rec.slot) & 0xffff);
                d.slot[2] = uint16_t(uint32_t(r.rec.slot) >> 16);
                d.k = 0;
                if (p.stages.size() + behind.size() >= 255) return QSIM_E_ARG;
                d.kx = uint8_t(p.stages.size() + behind.size());
                out->ops.push_back(d);
                dummy();
                DevOp l{};
                l.kind = DEVOP_LAYOUT;
                l.kx = d.kx;
                uint8_t *raw = reinterpret_cast<uint8_t *>(&l);
                for (int j = 0; j < 15; j++) {
                    const uint16_t v = uint16_t(j < t ? map_index(r.map, V[j]) : j < 14 ? 0 : r.map.c);
                    std::memcpy(raw + (j < 7 ? 2 * j : 16 + 2 * (j - 7)), &v, 2);
                }
                behind.push_back(l);
                if (r.rec.kind != DEVOP_RESET) grown = 0.0;   // scaled to norm 1
                continue;
            }
            const PauliOp &o = P.ops[size_t(idx)];
            DevOp d{};
            d.kind = DEVOP_PAULI;
            d.coef = uint32_t(out->coefs.size());
            if (!string_record(o.x, o.z, V, t, regs, &d)) return QSIM_E_ARG;
            if (o.two) {
                DevOp w{};
                if (!o.x || __builtin_popcountll(o.x & (o.z ^ o.z2)) & 1) return QSIM_E_ARG;
                if (!string_record(0, o.z ^ o.z2, V, t, regs, &w)) return QSIM_E_ARG;
                d.kind = DEVOP_PAULI2;
                w.kind = DEVOP_PAULI2X;
                w.k = 0;
                out->ops.push_back(d);
                const double a1 = kappa(o.x, o.z) * o.phi, a2 = kappa(o.x, o.z2) * o.phi2;
                out->coefs.push_back(branch_coefs(a1 + a2));
                out->coefs.push_back(branch_coefs(a1 - a2));
                out->op_np.push_back(0);
                for (int j = 0; j < 3; j++) out->op_slots.push_back(-1);
                for (int j = 0; j < 2; j++) {
                    out->ops.push_back(w);
                    dummy();
                }
                out->terms += 2;
                continue;
            }
            // y[i] = a x[i] + b (-1)^(i . z) x[i ^ x] with a = cos phi and
            // b = -i sin phi (-i)^ny, ny = |x & z|: t is its real or imaginary part
            const double k = kappa(o.x, o.z) * o.sign;
            out->ops.push_back(d);
            if (o.slot >= 0) {
                // bound per state: the sign of t (four entries of template)
                out->coefs.push_back(cd(k, 0.0));
                for (int j = 0; j < 3; j++) out->coefs.push_back(cd(0.0, 0.0));
                out->op_np.push_back(1);
                out->op_slots.push_back(o.slot);
            } else {
                cd e[2];
                pauli_coefs(std::cos(o.phi), k * std::sin(o.phi), single, e);
                grown += 0.5 * std::log2(1.0 + e[1].imag() * e[1].imag());
                if (grown > kGrownMost[single]) {
                    e[1] = cd(1.0, e[1].imag());
                    grown = 0.0;
                }
                out->coefs.push_back(e[0]);
                out->coefs.push_back(e[1]);
                out->op_np.push_back(0);
                out->op_slots.push_back(-1);
            }
            out->op_slots.push_back(-1);
            out->op_slots.push_back(-1);
            out->terms += o.x ? 2 : 1;
        }
    }
    *run = uint32_t(out->ops.size() - before);
    for (const DevOp &l : behind) {
        out->ops.push_back(l);
        dummy();
    }
    return QSIM_OK;
}

bool plan_expect(int n, int c, const qsim_pauli *terms, size_t nt, ExpectPlan *out) {
    const int t = std::min(n, 12), regs = kSpanRegs;
    out->t = t;
    out->recs.clear();
    out->groups.clear();
    out->max_rec = out->max_stage = 0;
    out->relaid = false;
    if (!span_tile_ok(t) || n > 48) return false;
    const uint64_t all = (uint64_t(1) << n) - 1;
    // the terms in ascending order of their X masks, and the identity (whose
    // value is the norm) first
    struct Term {
        uint64_t x, z;
        uint32_t k;
    };
    std::vector<Term> all_terms(nt + 1);
    for (size_t k = 0; k < nt; k++) all_terms[k] = {terms[k].xmask, terms[k].zmask, uint32_t(k)};
    all_terms[nt] = {0, 0, uint32_t(nt)};
    if (nt < 256) {
        std::sort(all_terms.begin(), all_terms.end(),
                  [](const Term &a, const Term &b) { return a.x != b.x ? a.x < b.x : a.k < b.k; });
    } else {
        // by digits of 11 bits, lowest first (3,000 terms: 30 us where sorting takes 155)
        std::vector<Term> by(nt + 1);
        for (int shift = 0; shift < n; shift += 11) {
            uint32_t at[2049] = {0};
            for (const Term &a : all_terms) at[((a.x >> shift) & 2047) + 1]++;
            for (int d = 0; d < 2048; d++) at[d + 1] += at[d];
            for (const Term &a : all_terms) by[at[(a.x >> shift) & 2047]++] = a;
            by.swap(all_terms);
        }
    }
    auto X = [&](uint32_t i) { return all_terms[i].x; };
    out->recs.reserve(2 * nt + 4);
    // (in blocks, so that planning stays linear in the number of terms)
    std::vector<uint32_t> left, later, sel, rest, mine;
    std::vector<uint64_t> dirs;
    constexpr int kMisses = 64;
    size_t taken = 0;
    while (taken < all_terms.size() || !left.empty()) {
        if (left.empty()) {
            const size_t end = std::min(all_terms.size(), taken + 2048);
            for (; taken < end; taken++) left.push_back(uint32_t(taken));
        }
        // a group: terms whose X masks lie in one tile's space
        Span T;
        for (int q = 0; q < std::min(c, t); q++) T.add(uint64_t(1) << q);
        later.clear();
        sel.clear();
        // (once the space is full, few of the others lie in it: the search ends after
        // kMisses in a row, or planning 3,000 masks would take longer than they do)
        size_t at = 0;
        for (int misses = 0; at < left.size() && sel.size() < kExpectGroup && misses < kMisses; at++) {
            const uint64_t r = T.reduce(X(left[at]));
            if (r == 0 || T.d < t) {
                if (r) T.add(r);
                sel.push_back(left[at]);
                misses = 0;
            } else {
                later.push_back(left[at]);
                misses++;
            }
        }
        later.insert(later.end(), left.begin() + long(at), left.end());
        left.swap(later);
        for (int q = 0; q < n && T.d < t; q++) {
            const uint64_t r = T.reduce(uint64_t(1) << q);
            if (r) T.add(r);
        }
        ExpectGroup g{};
        g.rest_mask = all & ~T.pm;
        g.rec_begin = uint32_t(out->recs.size());
        while (!sel.empty()) {
            // a stage: at most `regs` independent X masks
            Span R;
            dirs.clear();
            mine.clear();
            rest.clear();
            // (equal masks follow each other)
            for (size_t i = 0; i < sel.size(); i++) {
                const uint64_t x = X(sel[i]);
                const bool have = !x || (!dirs.empty() && dirs.back() == x);
                if (!have && R.d == regs) {
                    rest.insert(rest.end(), sel.begin() + long(i), sel.end());
                    break;
                }
                const uint64_t r = have ? 0 : R.reduce(x);
                if (have || r) {
                    if (r) {
                        R.add(r);
                        dirs.push_back(x);
                    }
                    mine.push_back(sel[i]);
                } else {
                    rest.push_back(sel[i]);
                }
            }
            sel.swap(rest);
            SpanStage st;
            stage_layout(T, dirs, t, c, regs, &st);
            uint64_t V[16];
            for (int j = 0; j < t; j++) {
                V[j] = 0;
                for (uint32_t m = st.layout[j]; m; m &= m - 1) V[j] ^= T.v[__builtin_ctz(m)];
                if (g.stages == 0) g.load_v[j] = V[j];
            }
            out->recs.push_back(stage_record(st, t, int(g.stages++)));
            for (uint32_t i : mine) {
                DevOp d{};
                d.kind = DEVOP_EXPECT;
                d.coef = all_terms[i].k;
                if (!string_record(all_terms[i].x, all_terms[i].z, V, t, regs, &d)) return false;
                out->recs.push_back(d);
            }
        }
        g.rec_end = uint32_t(out->recs.size());
        out->max_rec = std::max(out->max_rec, g.rec_end - g.rec_begin);
        out->max_stage = std::max(out->max_stage, g.stages);
        out->relaid = out->relaid || g.stages > 1;
        out->groups.push_back(g);
    }
    return true;
}

double expect_value(const qsim_pauli &t, double sum) {
    // <P> = sum over pairs {i, i ^ x} of 2 (-i)^ny s_i Re or i Im of conj(a_i) a_(i ^ x)
    if (!t.xmask) return sum;
    return (__builtin_popcountll(t.xmask & t.zmask) & 2) ? -2.0 * sum : 2.0 * sum;
}

}  // namespace qs
