// Index-notation front-end and leaf generator: statements of tensor index
// notation (Sec. II-A) over the library's level formats (Sec. II-B, III-B)
// are parsed, given a concordant loop order and lowered to HIP leaves in
// which each index variable is a coordinate-value loop or a co-iteration of
// the Compressed levels that index it (Sec. IV-C); sparse outputs are
// assembled in two phases (Sec. V-B).  See tin.hpp.
#include "tin.hpp"

#include <hip/hiprtc.h>

#include <algorithm>
#include <cctype>
#include <cstdint>
#include <cstdio>
#include <set>
#include <sstream>

#include "internal.hpp"

namespace spl {
namespace tin {
namespace {

// ------------------------------------------------------------------ syntax

struct Access {
    std::string name;
    std::vector<int> vars;
    int op = -1;  // binding index (right side)
};

struct Term {
    int sign = 1;
    std::vector<Access> f;
};

// lhs = sum of signed terms, each a product of accesses
struct Stmt {
    Access lhs;
    std::vector<Term> terms;
    std::vector<std::string> vars;
};

class Parser {
  public:
    Parser(const char *s, Stmt &st, std::string &err) : p_(s), st_(st), err_(err) {}

    bool parse() {
        if (!access(st_.lhs)) return false;
        if (!eat('=')) return fail("expected '='");
        int sign = 1;
        if (eat('-'))
            sign = -1;
        else
            eat('+');
        for (;;) {
            Term t;
            t.sign = sign;
            if (!term(t)) return false;
            st_.terms.push_back(t);
            if (eat('+'))
                sign = 1;
            else if (eat('-'))
                sign = -1;
            else
                break;
        }
        ws();
        if (*p_) return fail(std::string("unexpected '") + *p_ + "'");
        return true;
    }

  private:
    const char *p_;
    Stmt &st_;
    std::string &err_;

    bool fail(const std::string &m) {
        err_ = m;
        return false;
    }
    void ws() {
        while (*p_ && std::isspace(static_cast<unsigned char>(*p_))) ++p_;
    }
    bool eat(char c) {
        ws();
        if (*p_ != c) return false;
        ++p_;
        return true;
    }
    bool ident(std::string &s) {
        ws();
        if (!(std::isalpha(static_cast<unsigned char>(*p_)) || *p_ == '_')) return false;
        const char *b = p_;
        while (std::isalnum(static_cast<unsigned char>(*p_)) || *p_ == '_') ++p_;
        s.assign(b, p_);
        return true;
    }
    int var(const std::string &n) {
        for (size_t k = 0; k < st_.vars.size(); ++k)
            if (st_.vars[k] == n) return static_cast<int>(k);
        st_.vars.push_back(n);
        return static_cast<int>(st_.vars.size()) - 1;
    }
    bool access(Access &a) {
        if (!ident(a.name)) return fail("expected a tensor name");
        if (eat('(') && !eat(')')) {
            do {
                std::string v;
                if (!ident(v)) return fail("expected an index variable");
                a.vars.push_back(var(v));
            } while (eat(','));
            if (!eat(')')) return fail("expected ')'");
        }
        return true;
    }
    bool term(Term &t) {
        do {
            Access a;
            if (!access(a)) return false;
            t.f.push_back(a);
        } while (eat('*'));
        return true;
    }
};

// ------------------------------------------------------------- operands

struct OpInfo {
    bool sparse = false;
    int order = 0;
    int level[3] = {0, 0, 0};
    int dtype = 0;
    int64_t dims[3] = {0, 0, 0};
};

bool op_info(const Binding &b, OpInfo &o, std::string &err) {
    if ((b.sparse != nullptr) == (b.dense != nullptr)) {
        err = "operand " + b.name + ": bind exactly one of a sparse and a dense tensor";
        return false;
    }
    if (b.sparse) {
        const spl_sparse *s = b.sparse;
        o.sparse = true;
        o.order = s->order;
        o.dtype = s->vtype;
        for (int l = 0; l < s->order && l < 3; ++l) {
            o.level[l] = s->level[l];
            o.dims[l] = s->dims[l];
        }
        if (s->order < 2 || s->order > 3 || s->level[0] != SPL_DENSE ||
            s->level[s->order - 1] != SPL_COMPRESSED) {
            err = "operand " + b.name + ": formats (Dense, Compressed), (Dense, Compressed, "
                  "Compressed) or (Dense, Dense, Compressed)";
            return false;
        }
        if (s->pos_type != SPL_I32) {
            err = "operand " + b.name + ": int32 positions only";
            return false;
        }
    } else {
        const spl_dense *d = b.dense;
        o.order = d->ndim;
        o.dtype = d->dtype;
        o.dims[0] = d->dims[0];
        o.dims[1] = d->ndim == 2 ? d->dims[1] : 0;
        if (d->ndim != 1 && d->ndim != 2) {
            err = "operand " + b.name + ": dense operands are vectors or matrices";
            return false;
        }
    }
    return true;
}

// ------------------------------------------------------------- emission

struct Emitter {
    std::ostringstream s;
    int ind = 0;
    void line(const std::string &t) {
        for (int k = 0; k < ind; ++k) s << "    ";
        s << t << "\n";
    }
    void open(const std::string &t) {
        line(t);
        ++ind;
    }
    void close(const std::string &t = "}") {
        --ind;
        line(t);
    }
};

std::string join(const std::vector<std::string> &v, const std::string &sep) {
    std::string r;
    for (size_t k = 0; k < v.size(); ++k) r += (k ? sep : "") + v[k];
    return r;
}

std::string num(int64_t v) { return std::to_string(v); }

// Everything the code generator needs about one planned statement.
struct Gen {
    const Stmt &st;
    const std::vector<OpInfo> &oi;
    const OpInfo &out;
    int out_kind;
    std::vector<int> order;
    std::vector<int> slot_of_extent;  // per variable
    // per flattened access (terms in order, factors in order)
    std::vector<const Access *> acc;
    std::vector<int> acc_term;
    std::vector<int> acc_slot;        // first slot of the access
    std::string T;                    // value type
    int w = -1;                       // second output variable (dense 2-D, CSR)
    enum Mode { kEval, kCount, kFill } mode = kEval;
    // emitting the copy of the nest that reads the LDS stage (positions are
    // then relative to the workgroup's first ones, B<a>_1)
    mutable bool staged = false;

    std::string coord(int v) const { return "c" + num(v); }

    bool sparse(int a) const { return oi[acc[a]->op].sparse; }
    int last_level(int a) const { return oi[acc[a]->op].order - 1; }

    void emit_terms(Emitter &e, const std::string &target) const {
        for (size_t t = 0; t < st.terms.size(); ++t) {
            std::vector<std::string> guard, fac;
            for (size_t a = 0; a < acc.size(); ++a) {
                if (acc_term[a] != static_cast<int>(t)) continue;
                const Access &x = *acc[a];
                if (sparse(a)) {
                    const int L = last_level(a);
                    guard.push_back("h" + num(a) + "_" + num(L));
                    fac.push_back("(double)V" + num(a) + "[p" + num(a) + "_" + num(L) + "]");
                } else if (x.vars.size() == 1) {
                    fac.push_back("(double)D" + num(a) + "[" + coord(x.vars[0]) + "]");
                } else {
                    fac.push_back("(double)D" + num(a) + "[" + coord(x.vars[0]) + " * L" + num(a) +
                                  " + " + coord(x.vars[1]) + "]");
                }
            }
            const std::string val = (st.terms[t].sign < 0 ? "-(" : "(") + join(fac, " * ") + ")";
            if (guard.empty())
                e.line(target + " += " + val + ";");
            else
                e.line("if (" + join(guard, " && ") + ") " + target + " += " + val + ";");
        }
    }

    std::string body_target() const {
        if (out_kind == kOutScalar) return "tot";
        if (out_kind == kOutCsr) return "acc";
        if (w < 0) return "acc0";
        // dense 2-D: F64 outputs accumulate in place, F32 ones in F64 scratch
        if (T == "double") return "O[i0 * OL + " + coord(w) + "]";
        return "W[i0 * E" + num(w) + " + " + coord(w) + "]";
    }

    void emit_level(Emitter &e, size_t depth) const {
        if (depth == order.size()) {
            emit_terms(e, body_target());
            return;
        }
        const int v = order[depth];
        struct Part {
            int a, l;
        };
        std::vector<Part> parts, dlev;
        for (size_t a = 0; a < acc.size(); ++a) {
            if (!sparse(a)) continue;
            const OpInfo &o = oi[acc[a]->op];
            for (int l = 1; l < o.order; ++l)
                if (acc[a]->vars[l] == v)
                    (o.level[l] == SPL_COMPRESSED ? parts : dlev).push_back({static_cast<int>(a), l});
        }
        // a point of v counts when, for some term, every Compressed level of
        // that term's operands indexed by v stores it (union over terms,
        // intersection within a term); a term with no such level counts
        // every coordinate, so v is then iterated densely
        bool always = false;
        std::vector<std::vector<int>> conj(st.terms.size());
        for (size_t t = 0; t < st.terms.size(); ++t) {
            for (size_t k = 0; k < parts.size(); ++k)
                if (acc_term[parts[k].a] == static_cast<int>(t)) conj[t].push_back(static_cast<int>(k));
            if (conj[t].empty()) always = true;
        }
        auto P = [&](const Part &x) { return num(x.a) + "_" + num(x.l); };
        // the merge state of access a at level l: q, e, m suffixed a_l
        auto A = [&](const Part &x) { return num(x.a) + "_" + num(x.l); };
        for (const Part &x : parts) {
            const std::string par = num(x.a) + "_" + num(x.l - 1);
            const std::string at = "P" + P(x) + "[p" + par, off = staged ? " - B" + A(x) : "";
            if (staged)  // the outermost index always holds
                e.line("int q" + A(x) + " = " + at + "]" + off + "; const int e" + A(x) + " = " + at +
                       " + 1]" + off + ";");
            else
                e.line("i64 q" + A(x) + " = h" + par + " ? (i64)" + at + "] : 0, e" + A(x) + " = h" +
                       par + " ? (i64)" + at + " + 1] : 0;");
            head(e, "int ", A(x), P(x));
        }
        const std::string c = coord(v);
        std::vector<std::string> cond_terms;
        for (const auto &cj : conj) {
            std::vector<std::string> m;
            for (int k : cj) m.push_back("m" + A(parts[k]));
            cond_terms.push_back("(" + join(m, " && ") + ")");
        }
        if (always) {
            e.open("for (i64 " + c + " = 0; " + c + " < E" + num(v) + "; ++" + c + ") {");
            for (const Part &x : parts) e.line("const bool m" + A(x) + " = x" + A(x) + " == " + c + ";");
            descend(e, depth, parts, dlev);
            for (const Part &x : parts) advance(e, A(x), P(x));
            e.close();
            return;
        }
        std::vector<std::string> live;
        for (const Part &x : parts) live.push_back("q" + A(x) + " < e" + A(x));
        // one term: every level must store the point, so stop at the first
        // exhausted one; several: walk until all are exhausted
        e.open("while (" + join(live, st.terms.size() == 1 ? " && " : " || ") + ") {");
        std::string low = "x" + A(parts[0]);
        for (size_t k = 1; k < parts.size(); ++k) low = "min(" + low + ", x" + A(parts[k]) + ")";
        e.line("const i64 " + c + " = " + low + ";");
        for (const Part &x : parts) e.line("const bool m" + A(x) + " = x" + A(x) + " == " + c + ";");
        e.open("if (" + join(cond_terms, " || ") + ") {");
        descend(e, depth, parts, dlev);
        e.close();
        for (const Part &x : parts) advance(e, A(x), P(x));
        e.close();
    }

    // The coordinate at the head of a level's list, kept in a register:
    // 0x7fffffff (no coordinate reaches it) once the list is exhausted.  The
    // staged lists have a spare entry, so their heads are read without a
    // branch.
    void head(Emitter &e, const std::string &decl, const std::string &a, const std::string &p) const {
        if (staged) {
            if (!decl.empty()) e.line(decl + "x" + a + ";");
            e.line("{ const int h = C" + p + "[q" + a + "]; x" + a + " = q" + a + " < e" + a +
                   " ? h : 0x7fffffff; }");
        } else {
            e.line(decl + "x" + a + " = q" + a + " < e" + a + " ? C" + p + "[q" + a +
                   "] : 0x7fffffff;");
        }
    }
    void advance(Emitter &e, const std::string &a, const std::string &p) const {
        if (staged) {
            e.line("q" + a + " += m" + a + ";");
            head(e, "", a, p);
        } else {
            e.open("if (m" + a + ") {");
            e.line("++q" + a + ";");
            head(e, "", a, p);
            e.close();
        }
    }

    // Whether the count and fill kernels may stage their rows in LDS: every
    // sparse operand is a CSR matrix, so the rows of a workgroup own one run
    // of each operand's coordinates, and of the output's entries.
    bool stages() const {
        if (out_kind != kOutCsr) return false;
        for (size_t a = 0; a < acc.size(); ++a)
            if (sparse(a) && oi[acc[a]->op].order != 2) return false;
        return true;
    }
    // A sparse access merged into the output's rows (its lists are staged).
    bool merged(size_t a) const { return sparse(a) && acc[a]->vars[1] == w; }
    // Whether an entry's value depends on its row other than through the
    // merged positions.
    bool row_needed() const {
        for (size_t a = 0; a < acc.size(); ++a) {
            if (sparse(a) && !merged(a)) return true;
            if (!sparse(a) && acc[a]->vars[0] == order[0]) return true;
            if (!sparse(a) && acc[a]->vars.size() == 2 && acc[a]->vars[1] == order[0]) return true;
        }
        return false;
    }
    int entry_bytes() const {  // LDS bytes of one output entry in the fill's stage
        int b = 4 + (row_needed() ? 2 : 0);
        for (size_t a = 0; a < acc.size(); ++a) b += merged(a) ? 2 : 0;
        return b;
    }

    // The staged form of a count or fill kernel, for a workgroup whose runs
    // fit the LDS it was launched with.  The coordinate runs are copied in
    // with coalesced loads and a lane per row walks its lists there.  A fill
    // only notes each output entry's coordinate and the operands' positions
    // that meet there; then every lane takes one entry after another, works
    // out its value (neighbouring entries read neighbouring values) and
    // stores it beside its neighbours'.  A lane reading and storing its row
    // in HBM keeps a few lines per lane open, more than the caches hold: on
    // B - C of 1e6 rows (two F64 operands of 8 entries a row, 13.6 out) the
    // count took 103 us against 32 staged and the fill 751 against 117.
    // (Copying the values into the stage as well and the finished output out
    // of it: 265; values loaded entry by entry behind branches: 190.)  A
    // staged position fits 16 bits: the stage holds at most kStageBytes / 4.
    void emit_staged(Emitter &e, int pool_slot) const {
        e.line("extern __shared__ __attribute__((aligned(16))) char lds[];");
        e.line("const i64 g0 = (i64)blockIdx.x * blockDim.x, g1 = g0 + blockDim.x < n0 ? g0 + blockDim.x : n0;");
        std::string need = "(i64)0";
        for (size_t a = 0; a < acc.size(); ++a) {
            if (!merged(a)) continue;
            const std::string n = num(a) + "_1";
            e.line("const int B" + n + " = P" + n + "[g0], R" + n + " = P" + n + "[g1] - B" + n + ";");
            need += " + (i64)R" + n + " * 4 + 4";
        }
        if (mode == kFill) {
            e.line("const int BO = OP[g0], RO = OP[g1] - BO;");
            need += " + (i64)RO * " + num(entry_bytes());
        }
        e.open("if (" + need + " <= (i64)a.s[" + num(pool_slot) + "]) {");
        std::string at = "lds";
        for (size_t a = 0; a < acc.size(); ++a) {
            if (!merged(a)) continue;
            const std::string n = num(a) + "_1";
            e.line("int *sC" + n + " = (int *)(" + at + ");");
            at = "sC" + n + " + R" + n + " + 1";  // a spare entry
        }
        if (mode == kFill) {
            e.line("int *sOC = (int *)(" + at + ");");
            at = "sOC + RO";
            for (size_t a = 0; a < acc.size(); ++a) {
                if (!merged(a)) continue;
                e.line("unsigned short *sI" + num(a) + " = (unsigned short *)(" + at + ");");
                at = "sI" + num(a) + " + RO";
            }
            if (row_needed()) e.line("unsigned short *sR = (unsigned short *)(" + at + ");");
        }
        for (size_t a = 0; a < acc.size(); ++a) {
            if (!merged(a)) continue;
            const std::string n = num(a) + "_1";
            e.line("_Pragma(\"unroll 8\") for (int k = threadIdx.x; k < R" + n + "; k += blockDim.x) sC" + n +
                   "[k] = C" + n + "[B" + n + " + k];");
        }
        e.line("__syncthreads();");
        e.open("if (i0 < n0) {");
        for (size_t a = 0; a < acc.size(); ++a)
            if (merged(a)) e.line("const int *C" + num(a) + "_1 = sC" + num(a) + "_1;");
        e.line(mode == kCount ? "int cnt = 0;" : "int q = OP[i0] - BO;");
        staged = true;
        emit_level(e, 1);
        staged = false;
        if (mode == kCount) e.line("OP[i0 + 1] = cnt;");
        e.close();
        if (mode == kFill) {
            e.line("__syncthreads();");
            if (order.size() == 2) {
                emit_entries(e);
            } else {
                e.open("for (int k = threadIdx.x; k < RO; k += blockDim.x) {");
                e.line("const i64 " + coord(w) + " = sOC[k];");
                if (row_needed()) {
                    e.line("const i64 i0 = g0 + sR[k], " + coord(order[0]) + " = i0;");
                    for (size_t a = 0; a < acc.size(); ++a)
                        if (sparse(a) && !merged(a))
                            e.line("const i64 p" + num(a) + "_0 = i0; const bool h" + num(a) + "_0 = true;");
                }
                for (size_t a = 0; a < acc.size(); ++a) {
                    if (!merged(a)) continue;
                    const std::string n = num(a) + "_1";
                    e.line("const i64 p" + n + " = (i64)B" + n + " + sI" + num(a) + "[k]; const bool h" + n +
                           " = sI" + num(a) + "[k] != 0xffff;");
                }
                e.line("double acc = 0.0;");
                emit_level(e, 2);
                e.line("OC[BO + k] = (int)" + coord(w) + "; OV[BO + k] = (" + T + ")acc;");
                e.close();
            }
        }
        e.line("return;");
        e.close();
    }

    // The staged entries' values when no index is summed: kEntryBatch entries
    // per lane at a time, every value and dense factor loaded before the
    // first is used and without branches (an operand that does not store the
    // coordinate passes an offset past its buffer's range and reads 0, which
    // is not added).  Eight at a time: the whole call 224 us on the operands
    // above, against 228 with four and 235 with two; 219 with the entries
    // stored past the caches.
    static constexpr int kEntryBatch = 8;
    void emit_entries(Emitter &e) const {
        const std::string U = num(kEntryBatch);
        const auto each = [&] { e.open("_Pragma(\"unroll\") for (int u = 0; u < " + U + "; ++u) {"); };
        for (size_t a = 0; a < acc.size(); ++a)
            if (merged(a))
                e.line("const auto rV" + num(a) + " = __builtin_amdgcn_make_buffer_rsrc((void *)(V" + num(a) +
                       " + B" + num(a) + "_1), 0, R" + num(a) + "_1 * (int)sizeof(" + T + "), 0x00020000);");
        e.open("for (int k0 = threadIdx.x; k0 < RO; k0 += " + U + " * blockDim.x) {");
        e.line("int cw[" + U + "];" + (row_needed() ? " i64 ci[" + U + "];" : ""));
        for (size_t a = 0; a < acc.size(); ++a) {
            if (merged(a)) e.line("bool f" + num(a) + "[" + U + "];");
            e.line(T + " v" + num(a) + "[" + U + "];");
        }
        each();
        e.line("const int k = k0 + u * (int)blockDim.x, kk = k < RO ? k : RO - 1;");
        e.line("cw[u] = sOC[kk];");
        if (row_needed()) e.line("ci[u] = g0 + sR[kk];");
        for (size_t a = 0; a < acc.size(); ++a) {
            if (!merged(a)) continue;
            const std::string n = num(a);
            e.line("{ const int s = sI" + n + "[kk]; f" + n + "[u] = s != 0xffff; v" + n + "[u] = load_" + T +
                   "(rV" + n + ", f" + n + "[u] ? s * (int)sizeof(" + T + ") : -16); }");
        }
        e.close();
        each();
        for (size_t a = 0; a < acc.size(); ++a) {
            if (merged(a)) continue;
            auto at = [&](int v) { return std::string(v == order[0] ? "ci[u]" : "(i64)cw[u]"); };
            const Access &x = *acc[a];
            e.line("v" + num(a) + "[u] = D" + num(a) + "[" + at(x.vars[0]) +
                   (x.vars.size() == 2 ? " * L" + num(a) + " + " + at(x.vars[1]) : std::string()) + "];");
        }
        e.close();
        each();
        e.line("const int k = k0 + u * (int)blockDim.x;");
        e.line("double acc = 0.0;");
        for (size_t t = 0; t < st.terms.size(); ++t) {
            std::vector<std::string> guard, fac;
            for (size_t a = 0; a < acc.size(); ++a) {
                if (acc_term[a] != static_cast<int>(t)) continue;
                if (merged(a)) guard.push_back("f" + num(a) + "[u]");
                fac.push_back("(double)v" + num(a) + "[u]");
            }
            const std::string sum = std::string("acc + ") + (st.terms[t].sign < 0 ? "-(" : "(") +
                                    join(fac, " * ") + ")";
            e.line("acc = " + (guard.empty() ? sum : "(" + join(guard, " && ") + ") ? " + sum + " : acc") + ";");
        }
        e.line("if (k < RO) { __builtin_nontemporal_store(cw[u], OC + BO + k); __builtin_nontemporal_store((" + T + ")acc, OV + BO + k); }");
        e.close();
        e.close();
    }

    template <typename PartT>
    void descend(Emitter &e, size_t depth, const std::vector<PartT> &parts,
                 const std::vector<PartT> &dlev) const {
        const int v = order[depth];
        for (const auto &x : parts) {
            const std::string n = num(x.a) + "_" + num(x.l);
            e.line("const i64 p" + n + " = q" + n + "; const bool h" + n + " = m" + n + ";");
        }
        for (const auto &x : dlev) {
            const std::string n = num(x.a) + "_" + num(x.l), par = num(x.a) + "_" + num(x.l - 1);
            e.line("const i64 p" + n + " = p" + par + " * N" + n + " + " + coord(v) +
                   "; const bool h" + n + " = h" + par + ";");
        }
        if (out_kind == kOutCsr && depth == 1) {
            // the second output coordinate is emitted here
            if (mode == kCount) {
                e.line("++cnt;");
                return;
            }
            if (staged) {
                e.line("sOC[q] = (int)" + coord(v) + ";");
                for (size_t a = 0; a < acc.size(); ++a)
                    if (merged(a))
                        e.line("sI" + num(a) + "[q] = (unsigned short)(h" + num(a) + "_1 ? p" + num(a) +
                               "_1 : 0xffff);");
                if (row_needed()) e.line("sR[q] = (unsigned short)threadIdx.x;");
                e.line("++q;");
                return;
            }
            e.line("double acc = 0.0;");
            emit_level(e, depth + 1);
            e.line("OC[q] = (int)" + coord(v) + "; OV[q] = (" + T + ")acc; ++q;");
            return;
        }
        emit_level(e, depth + 1);
    }

    std::string kernel(const std::string &name) const {
        Emitter e;
        e.open("extern \"C\" __global__ void __launch_bounds__(256) " + name + "(TinArgs a) {");
        e.line("const i64 i0 = (i64)blockIdx.x * blockDim.x + threadIdx.x;");
        e.line("const i64 n0 = (i64)a.s[0];");
        const bool stage = stages();
        if (!stage) e.line("if (i0 >= n0) return;");
        for (size_t v = 0; v < st.vars.size(); ++v)
            e.line("const i64 E" + num(v) + " = (i64)a.s[" + num(slot_of_extent[v]) + "];");
        for (size_t a = 0; a < acc.size(); ++a) {
            int k = acc_slot[a];
            const OpInfo &o = oi[acc[a]->op];
            if (o.sparse) {
                for (int l = 1; l < o.order; ++l) {
                    const std::string n = num(a) + "_" + num(l);
                    if (o.level[l] == SPL_COMPRESSED) {
                        e.line("const int *__restrict__ P" + n + " = (const int *)a.s[" + num(k++) + "];");
                        e.line("const int *__restrict__ C" + n + " = (const int *)a.s[" + num(k++) + "];");
                    } else {
                        e.line("const i64 N" + n + " = (i64)a.s[" + num(k++) + "];");
                    }
                }
                e.line("const " + T + " *__restrict__ V" + num(a) + " = (const " + T + " *)a.s[" + num(k++) + "];");
            } else {
                e.line("const " + T + " *__restrict__ D" + num(a) + " = (const " + T + " *)a.s[" + num(k++) + "];");
                e.line("const i64 L" + num(a) + " = (i64)a.s[" + num(k++) + "];");
            }
        }
        const int os = out_slot;
        const std::string c0 = coord(order[0]);
        e.line("const i64 " + c0 + " = i0;");
        for (size_t a = 0; a < acc.size(); ++a)
            if (sparse(a)) e.line("const i64 p" + num(a) + "_0 = i0; const bool h" + num(a) + "_0 = true;");
        if (out_kind == kOutScalar) {
            e.line("double *__restrict__ PART = (double *)a.s[" + num(os) + "];");
            e.line("double tot = 0.0;");
            emit_level(e, 1);
            e.line("PART[i0] = tot;");
        } else if (out_kind == kOutCsr) {
            e.line("int *__restrict__ OP = (int *)a.s[" + num(os) + "];");
            if (mode == kFill) {
                e.line("int *__restrict__ OC = (int *)a.s[" + num(os + 1) + "];");
                e.line(T + " *__restrict__ OV = (" + T + " *)a.s[" + num(os + 2) + "];");
            }
            if (stage) {
                emit_staged(e, os + 3);
                e.line("if (i0 >= n0) return;");
            }
            if (mode == kCount) {
                e.line("i64 cnt = 0;");
                emit_level(e, 1);
                e.line("OP[i0 + 1] = (int)cnt;");
            } else {
                e.line("i64 q = OP[i0];");
                emit_level(e, 1);
            }
        } else {
            e.line(T + " *__restrict__ O = (" + T + " *)a.s[" + num(os) + "];");
            e.line("const i64 OL = (i64)a.s[" + num(os + 1) + "];");
            if (w < 0) {
                e.line("double acc0 = 0.0;");
                emit_level(e, 1);
                e.line("O[i0] = (" + T + ")acc0;");
            } else if (T == "double") {
                e.line("for (i64 z = 0; z < E" + num(w) + "; ++z) O[i0 * OL + z] = 0.0;");
                emit_level(e, 1);
            } else {
                e.line("double *__restrict__ W = (double *)a.s[" + num(os + 2) + "];");
                e.line("for (i64 z = 0; z < E" + num(w) + "; ++z) W[i0 * E" + num(w) + " + z] = 0.0;");
                emit_level(e, 1);
                e.line("for (i64 z = 0; z < E" + num(w) + "; ++z) O[i0 * OL + z] = (float)W[i0 * E" +
                       num(w) + " + z];");
            }
        }
        e.close();
        return e.s.str();
    }

    int out_slot = 0;
};

}  // namespace

Program::~Program() {
    if (module) (void)hipModuleUnload(module);
}

spl_status plan(const char *stmt, const std::vector<Binding> &ops, const Binding &out,
                bool source, Program &prog, std::string &err) {
    if (!stmt) {
        err = "statement is NULL";
        return SPL_ERR_ARG;
    }
    Stmt st;
    Parser ps(stmt, st, err);
    if (!ps.parse()) {
        err = "index notation: " + err;
        return SPL_ERR_ARG;
    }
    // bind names
    std::vector<OpInfo> oi(ops.size());
    for (size_t k = 0; k < ops.size(); ++k) {
        if (!op_info(ops[k], oi[k], err)) return SPL_ERR_FORMAT;
        for (size_t m = 0; m < k; ++m)
            if (ops[m].name == ops[k].name) {
                err = "operand " + ops[k].name + " bound twice";
                return SPL_ERR_ARG;
            }
    }
    if (out.name != st.lhs.name) {
        err = "the output is bound as " + out.name + " but the statement assigns " + st.lhs.name;
        return SPL_ERR_ARG;
    }
    OpInfo oo;
    if (!op_info(out, oo, err)) return SPL_ERR_FORMAT;
    std::set<int> first_set;
    bool first = true;
    for (Term &t : st.terms) {
        std::set<int> vs;
        for (Access &a : t.f) {
            if (a.name == st.lhs.name) {
                err = "the output " + a.name + " appears on the right side";
                return SPL_ERR_ARG;
            }
            for (size_t k = 0; k < ops.size(); ++k)
                if (ops[k].name == a.name) a.op = static_cast<int>(k);
            if (a.op < 0) {
                err = "operand " + a.name + " is not bound";
                return SPL_ERR_ARG;
            }
            if (static_cast<int>(a.vars.size()) != oi[a.op].order) {
                err = "operand " + a.name + " has order " + std::to_string(oi[a.op].order) +
                      " but is indexed by " + std::to_string(a.vars.size()) + " variables";
                return SPL_ERR_SHAPE;
            }
            std::set<int> own(a.vars.begin(), a.vars.end());
            if (own.size() != a.vars.size()) {
                err = "operand " + a.name + " repeats an index variable";
                return SPL_ERR_UNSUPPORTED;
            }
            vs.insert(a.vars.begin(), a.vars.end());
        }
        if (!first && vs != first_set) {
            err = "every term of a sum must use the same index variables";
            return SPL_ERR_UNSUPPORTED;
        }
        first_set = vs;
        first = false;
    }
    {
        std::set<int> own(st.lhs.vars.begin(), st.lhs.vars.end());
        if (own.size() != st.lhs.vars.size()) {
            err = "the output repeats an index variable";
            return SPL_ERR_UNSUPPORTED;
        }
        for (int v : st.lhs.vars)
            if (!first_set.count(v)) {
                err = "output variable " + st.vars[v] + " does not appear on the right side";
                return SPL_ERR_ARG;
            }
    }
    // value types
    const int vt = oi.empty() ? SPL_F64 : oi[0].dtype;
    if (vt != SPL_F64 && vt != SPL_F32) {
        err = "generated leaves take F64 or F32 values";
        return SPL_ERR_DTYPE;
    }
    for (const OpInfo &o : oi)
        if (o.dtype != vt) {
            err = "every operand must have the same value type";
            return SPL_ERR_DTYPE;
        }
    // output kind
    int kind;
    if (st.lhs.vars.empty()) {
        kind = kOutScalar;
        if (oo.sparse || oo.order != 1 || oo.dims[0] != 1 || oo.dtype != SPL_F64) {
            err = "a scalar output is a dense F64 vector of one entry";
            return SPL_ERR_SHAPE;
        }
    } else if (oo.sparse) {
        kind = kOutCsr;
        if (oo.order != 2 || oo.level[1] != SPL_COMPRESSED || st.lhs.vars.size() != 2) {
            err = "a sparse output is a CSR matrix (Dense, Compressed)";
            return SPL_ERR_FORMAT;
        }
        if (oo.dtype != vt) {
            err = "the output's value type must match the operands'";
            return SPL_ERR_DTYPE;
        }
    } else {
        kind = kOutDense;
        if (oo.order != static_cast<int>(st.lhs.vars.size())) {
            err = "the dense output's order does not match the statement";
            return SPL_ERR_SHAPE;
        }
        if (oo.dtype != vt) {
            err = "the output's value type must match the operands'";
            return SPL_ERR_DTYPE;
        }
    }
    // extents
    const int nv = static_cast<int>(st.vars.size());
    std::vector<int64_t> ext(nv, -1);
    auto set_ext = [&](int v, int64_t d, const std::string &who) {
        if (ext[v] < 0) ext[v] = d;
        if (ext[v] != d) {
            err = "index " + st.vars[v] + " has extent " + std::to_string(ext[v]) + " but " + who +
                  " gives " + std::to_string(d);
            return false;
        }
        return true;
    };
    for (const Term &t : st.terms)
        for (const Access &a : t.f)
            for (size_t l = 0; l < a.vars.size(); ++l)
                if (!set_ext(a.vars[l], oi[a.op].dims[l], a.name)) return SPL_ERR_SHAPE;
    for (size_t l = 0; l < st.lhs.vars.size(); ++l)
        if (!set_ext(st.lhs.vars[l], oo.dims[l], st.lhs.name)) return SPL_ERR_SHAPE;
    for (int v = 0; v < nv; ++v)
        if (ext[v] < 0 || ext[v] > 2147483647LL) {
            err = "index " + st.vars[v] + " has no usable extent";
            return SPL_ERR_SHAPE;
        }
    // the outermost index: the first of every sparse operand (their Dense
    // first level), one thread per coordinate
    int i0 = -1;
    for (const Term &t : st.terms)
        for (const Access &a : t.f)
            if (oi[a.op].sparse) {
                if (i0 < 0) i0 = a.vars[0];
                if (a.vars[0] != i0) {
                    err = "every sparse operand must be indexed first by the same variable";
                    return SPL_ERR_UNSUPPORTED;
                }
            }
    if (i0 < 0) i0 = st.lhs.vars.empty() ? st.terms[0].f[0].vars[0] : st.lhs.vars[0];
    if (!st.lhs.vars.empty() && st.lhs.vars[0] != i0) {
        err = "the output's first index must be the sparse operands' first (each thread owns "
              "one output row)";
        return SPL_ERR_UNSUPPORTED;
    }
    // concordant loop order: a sparse operand's level l needs its levels
    // before l outside it
    std::vector<std::set<int>> need(nv);
    bool uses_sparse[64] = {};
    if (nv > 64) {
        err = "too many index variables";
        return SPL_ERR_UNSUPPORTED;
    }
    for (const Term &t : st.terms)
        for (const Access &a : t.f)
            if (oi[a.op].sparse)
                for (size_t l = 0; l < a.vars.size(); ++l) {
                    uses_sparse[a.vars[l]] = true;
                    for (size_t m = 0; m < l; ++m) need[a.vars[l]].insert(a.vars[m]);
                }
    std::vector<int> order{i0};
    std::vector<bool> placed(nv, false);
    placed[i0] = true;
    const int w = st.lhs.vars.size() == 2 ? st.lhs.vars[1] : -1;
    while (static_cast<int>(order.size()) < nv) {
        int best = -1, best_rank = 1 << 30;
        for (int v = 0; v < nv; ++v) {
            if (placed[v]) continue;
            bool ready = true;
            for (int u : need[v]) ready = ready && placed[u];
            if (!ready) continue;
            // sparse output: its second index next; then the variables of
            // sparse levels; dense-only variables innermost
            int rank = (kind == kOutCsr && v == w) ? 0 : uses_sparse[v] ? 1 : 2;
            if (rank < best_rank) {
                best = v;
                best_rank = rank;
            }
        }
        if (best < 0) {
            err = "the sparse operands' level orders admit no common loop order";
            return SPL_ERR_UNSUPPORTED;
        }
        order.push_back(best);
        placed[best] = true;
    }
    if (kind == kOutCsr && order[1] != w) {
        err = "a sparse output's second index must be iterated right after its first";
        return SPL_ERR_UNSUPPORTED;
    }
    // slots and code
    Gen g{st, oi, oo, kind};
    g.order = order;
    g.T = vt == SPL_F64 ? "double" : "float";
    g.w = w;
    prog.slots.clear();
    prog.slots.push_back({Slot::kRows, -1, i0});
    g.slot_of_extent.resize(nv);
    for (int v = 0; v < nv; ++v) {
        g.slot_of_extent[v] = static_cast<int>(prog.slots.size());
        prog.slots.push_back({Slot::kExtent, -1, v});
    }
    for (size_t t = 0; t < st.terms.size(); ++t)
        for (const Access &a : st.terms[t].f) {
            g.acc.push_back(&a);
            g.acc_term.push_back(static_cast<int>(t));
            g.acc_slot.push_back(static_cast<int>(prog.slots.size()));
            const OpInfo &o = oi[a.op];
            if (o.sparse) {
                for (int l = 1; l < o.order; ++l) {
                    if (o.level[l] == SPL_COMPRESSED) {
                        prog.slots.push_back({Slot::kPos, a.op, l});
                        prog.slots.push_back({Slot::kCrd, a.op, l});
                    } else {
                        prog.slots.push_back({Slot::kLevelDim, a.op, l});
                    }
                }
                prog.slots.push_back({Slot::kVals, a.op, 0});
            } else {
                prog.slots.push_back({Slot::kDenseData, a.op, 0});
                prog.slots.push_back({Slot::kDenseLd, a.op, 0});
            }
        }
    g.out_slot = static_cast<int>(prog.slots.size());
    if (kind == kOutScalar) {
        prog.slots.push_back({Slot::kPartials, -1, 0});
    } else if (kind == kOutCsr) {
        prog.slots.push_back({Slot::kOutPos, -1, 0});
        prog.slots.push_back({Slot::kOutCrd, -1, 0});
        prog.slots.push_back({Slot::kOutVals, -1, 0});
        prog.slots.push_back({Slot::kPool, -1, 0});
    } else {
        prog.slots.push_back({Slot::kOutData, -1, 0});
        prog.slots.push_back({Slot::kOutLd, -1, 0});
        if (w >= 0 && vt == SPL_F32) prog.slots.push_back({Slot::kScratch, -1, 0});
    }
    if (prog.slots.size() > 120) {
        err = "statement too large";
        return SPL_ERR_UNSUPPORTED;
    }

    if (source) {
        std::ostringstream src;
        src << "// generated from: " << stmt << "\n";
        src << "typedef long long i64;\n";
        src << "struct TinArgs { unsigned long long s[" << prog.slots.size() << "]; };\n";
        if (g.stages())  // a value at a byte offset of a buffer; 0 past its range
            src << "__device__ __forceinline__ float load_float(__amdgpu_buffer_rsrc_t r, int off) {\n"
                   "    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));\n}\n"
                   "typedef unsigned u32x2 __attribute__((ext_vector_type(2)));\n"
                   "__device__ __forceinline__ double load_double(__amdgpu_buffer_rsrc_t r, int off) {\n"
                   "    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);\n"
                   "    return __hiloint2double((int)w[1], (int)w[0]);\n}\n";
        if (kind == kOutCsr) {
            g.mode = Gen::kCount;
            src << g.kernel("tin_count");
            g.mode = Gen::kFill;
            src << g.kernel("tin_fill");
        } else {
            g.mode = Gen::kEval;
            src << g.kernel("tin_eval");
        }
        prog.source = src.str();
    }
    prog.out_kind = kind;
    prog.vtype = vt;
    prog.rows = ext[i0];
    prog.extents = ext;
    prog.out_cols = w >= 0 ? ext[w] : 1;
    prog.scratch_rows = kind == kOutDense && w >= 0 && vt == SPL_F32;
    prog.stages = g.stages();
    prog.staged_ops.clear();
    prog.entry_bytes = prog.stages ? g.entry_bytes() : 0;
    if (prog.stages)
        for (size_t a = 0; a < g.acc.size(); ++a)
            if (g.merged(a)) prog.staged_ops.push_back(g.acc[a]->op);
    // the cache key: the statement and every operand's format, dtype and
    // shape (the shapes are runtime slots, but they are checked above)
    std::ostringstream key;
    key << stmt << "|" << out.name << ":" << oo.sparse << oo.order << oo.level[1] << oo.dtype;
    for (size_t k = 0; k < ops.size(); ++k)
        key << "|" << ops[k].name << ":" << oi[k].sparse << oi[k].order << oi[k].level[0]
            << oi[k].level[1] << oi[k].level[2] << oi[k].dtype;
    prog.key = key.str();
    return SPL_OK;
}

spl_status compile(Program &prog, std::string &err) {
    hiprtcProgram p = nullptr;
    if (hiprtcCreateProgram(&p, prog.source.c_str(), "tin.hip", 0, nullptr, nullptr) !=
        HIPRTC_SUCCESS) {
        err = "hiprtcCreateProgram failed";
        return SPL_ERR_HIP;
    }
    // no packed FP32 instructions in generated code either
    const char *opts[] = {"--offload-arch=gfx950", "-O3", "-Xclang", "-target-feature", "-Xclang",
                          "-packed-fp32-ops"};
    const hiprtcResult r = hiprtcCompileProgram(p, 6, opts);
    if (r != HIPRTC_SUCCESS) {
        size_t n = 0;
        hiprtcGetProgramLogSize(p, &n);
        std::string log(n + 1, '\0');
        if (n) hiprtcGetProgramLog(p, &log[0]);
        err = "generated leaf did not compile: " + log;
        hiprtcDestroyProgram(&p);
        return SPL_ERR_HIP;
    }
    size_t n = 0;
    hiprtcGetCodeSize(p, &n);
    std::vector<char> code(n);
    hiprtcGetCode(p, code.data());
    hiprtcDestroyProgram(&p);
    hipError_t e = hipModuleLoadData(&prog.module, code.data());
    if (e != hipSuccess) {
        (void)hipGetLastError();
        prog.module = nullptr;
        err = std::string("hipModuleLoadData: ") + hipGetErrorString(e);
        return SPL_ERR_HIP;
    }
    auto get = [&](const char *name, hipFunction_t &f) {
        hipError_t x = hipModuleGetFunction(&f, prog.module, name);
        if (x != hipSuccess) {
            (void)hipGetLastError();
            err = std::string("hipModuleGetFunction(") + name + "): " + hipGetErrorString(x);
            return false;
        }
        return true;
    };
    if (prog.out_kind == kOutCsr) {
        if (!get("tin_count", prog.f_count) || !get("tin_fill", prog.f_fill)) return SPL_ERR_HIP;
    } else if (!get("tin_eval", prog.f_eval)) {
        return SPL_ERR_HIP;
    }
    return SPL_OK;
}

void fill_slots(const Program &prog, const std::vector<Binding> &ops, const Binding &out,
                const int32_t *out_pos, void *partials, void *scratch, unsigned pool,
                std::vector<unsigned long long> &slots) {
    auto u = [](const void *p) { return static_cast<unsigned long long>(reinterpret_cast<uintptr_t>(p)); };
    slots.assign(prog.slots.size(), 0);
    for (size_t k = 0; k < prog.slots.size(); ++k) {
        const Slot &s = prog.slots[k];
        const Binding *b = s.operand >= 0 ? &ops[s.operand] : &out;
        switch (s.kind) {
        case Slot::kRows: slots[k] = static_cast<unsigned long long>(prog.rows); break;
        case Slot::kExtent: slots[k] = static_cast<unsigned long long>(prog.extents[s.level]); break;
        case Slot::kPos: slots[k] = u(b->sparse->pos[s.level]); break;
        case Slot::kCrd: slots[k] = u(b->sparse->crd[s.level]); break;
        case Slot::kVals: slots[k] = u(b->sparse->vals); break;
        case Slot::kLevelDim:
            slots[k] = static_cast<unsigned long long>(b->sparse->dims[s.level]);
            break;
        case Slot::kDenseData: slots[k] = u(b->dense->data); break;
        case Slot::kDenseLd: slots[k] = static_cast<unsigned long long>(b->dense->ld); break;
        case Slot::kOutData: slots[k] = u(out.dense->data); break;
        case Slot::kOutLd: slots[k] = static_cast<unsigned long long>(out.dense->ld); break;
        case Slot::kOutPos: slots[k] = u(out_pos); break;
        case Slot::kOutCrd: slots[k] = out.sparse ? u(out.sparse->crd[1]) : 0; break;
        case Slot::kOutVals: slots[k] = out.sparse ? u(out.sparse->vals) : 0; break;
        case Slot::kPartials: slots[k] = u(partials); break;
        case Slot::kScratch: slots[k] = u(scratch); break;
        case Slot::kPool: slots[k] = pool; break;
        }
    }
}

void stage_shape(const Program &prog, const std::vector<Binding> &ops, int64_t out_nnz,
                 unsigned &block, unsigned &pool) {
    block = 256;
    pool = 0;
    if (!prog.stages || prog.rows == 0) return;
    // expected bytes of one row's runs
    double bytes = out_nnz < 0 ? 0.0 : static_cast<double>(prog.entry_bytes) * static_cast<double>(out_nnz);
    for (int k : prog.staged_ops) bytes += 4.0 * static_cast<double>(ops[k].sparse->nnz);
    bytes /= static_cast<double>(prog.rows);
    const double room = kStageBytes - kStageSlack;
    for (unsigned b : {kStageRows, 64u}) {
        if (bytes * b * kStageSpread > room) continue;
        block = b;
        pool = static_cast<unsigned>(bytes * b * kStageSpread) + kStageSlack;
        pool = (pool + 1023u) & ~1023u;
        return;
    }
}

size_t workspace_bytes(const Program &prog, bool symbolic) {
    auto up = [](size_t v) { return (v + 255) & ~static_cast<size_t>(255); };
    const size_t rows = static_cast<size_t>(prog.rows);
    size_t b = 0;
    if (prog.out_kind == kOutScalar) b += up(rows * 8);
    if (prog.scratch_rows) b += up(rows * static_cast<size_t>(prog.out_cols) * 8);
    if (symbolic) b += up(static_cast<size_t>(spadd3_scan_tiles(prog.rows)) * 8) + up(8);
    return b;
}

}  // namespace tin
}  // namespace spl
