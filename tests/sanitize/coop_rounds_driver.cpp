// A model of the rounds of coop.hip on the CPU, over the library's own layout
// of the slices (csrc/prep.cpp) and slots (csrc/coop_rounds.h): workgroups
// that post and wait, one store or one load at a time, held up at any place
// for as long as the others can go on.  A workgroup that finds a later
// round's number where it waits for its own waits for ever; one that is two
// rounds ahead of another could write what that one still reads.  Exits
// non-zero if either happens, or if a layout leaves a workgroup without a
// slice or a row without an owner -- and if the model does not find the
// fault in layouts that have it (no empty slices, with the Q and A rounds'
// slots in common or apart).
#include <cstdio>
#include <random>
#include <vector>

#include "prep.h"

using namespace pdhcg;

namespace {

struct Program {                // the rounds of some iterations, the same in every workgroup
    std::vector<char> kind;     // 'Q' or 'A'
    std::vector<int> iter;
};

// right-hand side, inner steps of two rounds (some with one more), x_bar, the rows of A
Program program(std::mt19937& rng, int iters)
{
    Program p;
    for (int i = 0; i < iters; ++i) {
        const int q = 2 + (int)(rng() % 4) * 2 + (int)(rng() % 2);
        for (int r = 0; r < q; ++r) { p.kind.push_back('Q'); p.iter.push_back(i); }
        p.kind.push_back('A');
        p.iter.push_back(i);
    }
    return p;
}

struct Model {
    int W, nq, na, nslots;
    bool apart;                 // the A rounds' slots are of their own, alternating with the iteration
    const Program* p;
    std::vector<unsigned> slot;
    struct Wg { int round = 0, at = 0; bool waits = false; };
    std::vector<Wg> wg;
    bool overrun = false, lead = false;

    Model(int W_, int nq_, int na_, bool apart_, const Program* p_)
        : W(W_), nq(nq_), na(na_), nslots(nq_ > na_ ? nq_ : na_), apart(apart_), p(p_),
          slot((size_t)4 * nslots + 1, 0u), wg((size_t)W_)
    {
        for (int i = 0; i < W; ++i) wg[i].at = i;
    }
    int slices(int r) const { return p->kind[r] == 'Q' ? nq : na; }
    size_t where(int r, int s) const
    {
        const unsigned tag = (unsigned)r + 1u;
        if (apart && p->kind[r] == 'A') return (size_t)2 * nslots + coop_slot((unsigned)p->iter[r], nslots, s) / 8;
        return coop_slot(tag, nslots, s) / 8;
    }
    bool finished(int i) const { return wg[i].round == (int)p->kind.size(); }
    // one store or load of workgroup i; false if it cannot go on
    bool step(int i)
    {
        Wg& g = wg[i];
        if (finished(i)) return false;
        const int r = g.round, n = slices(r);
        if (!g.waits) {
            if (g.at < n) { slot[where(r, g.at)] = (unsigned)r + 1u; g.at += W; }
            else { g.waits = true; g.at = 0; }
            return true;
        }
        if (g.at < n) {
            const unsigned v = slot[where(r, g.at)];
            if (v > (unsigned)r + 1u) overrun = true;
            if (v != (unsigned)r + 1u) return false;
            ++g.at;
            return true;
        }
        g.waits = false;
        ++g.round;
        g.at = i;
        for (const Wg& o : wg)
            if (g.round - o.round > 1) lead = true;
        return true;
    }
    // everyone but `held` (-1: nobody) as far as they get; false if nobody moved
    bool run(int held, std::mt19937& rng)
    {
        bool any = false;
        for (bool moved = true; moved && !overrun;) {
            moved = false;
            const int first = (int)(rng() % (unsigned)W);
            for (int k = 0; k < W; ++k) {
                const int i = (first + k) % W;
                if (i == held) continue;
                for (unsigned steps = 1 + rng() % 40; steps > 0 && step(i); --steps) moved = any = true;
            }
        }
        return any;
    }
    bool all_finished() const
    {
        for (int i = 0; i < W; ++i)
            if (!finished(i)) return false;
        return true;
    }
};

// true if the rounds come to an end whatever workgroup is held up wherever
bool sound(int W, int nq, int na, bool apart, std::mt19937& rng)
{
    const Program p = program(rng, 3);
    for (int held = 0; held < W; held += 1 + W / 6)
        for (int r = 0; r < (int)p.kind.size(); ++r)
            for (int place = 0; place < 3; ++place) {   // before its post, before its first load, in the middle of them
                Model m(W, nq, na, apart, &p);
                // held reaches its place with the others' help, then they go on alone
                const int reads = place == 2 ? m.slices(r) / 2 : 0;
                auto there = [&] {
                    const Model::Wg& g = m.wg[held];
                    return g.round > r || (g.round == r && (place == 0 || (g.waits && g.at >= reads)));
                };
                while (!there() && !m.overrun) {
                    if (m.step(held)) continue;
                    // one workgroup that can move moves by one
                    bool moved = false;
                    const int first = (int)(rng() % (unsigned)W);
                    for (int k = 0; k < W && !moved; ++k) {
                        const int i = (first + k) % W;
                        moved = i != held && m.step(i);
                    }
                    if (!moved) break;
                }
                m.run(held, rng);
                m.run(-1, rng);
                if (m.overrun || m.lead || !m.all_finished()) return false;
            }
    return true;
}

int expect(const char* what, long long n, long long rows, int W, bool ok)
{
    if (!ok) std::printf("FAILED: %s (n = %lld, m = %lld, %d workgroups)\n", what, n, rows, W);
    return ok ? 0 : 1;
}

std::vector<int64_t> rowptr(int64_t rows, int64_t per)
{
    std::vector<int64_t> rp((size_t)rows + 1, 0);
    for (int64_t i = 0; i < rows; ++i) rp[i + 1] = rp[i] + per + (per > 1 ? i % 3 : 0);
    return rp;
}

int covers(const std::vector<BlkDesc>& s, const std::vector<int64_t>& rp, int threads)
{
    int64_t row = 0;
    int bad = 0;
    for (const BlkDesc& b : s) {
        if (b.nrows == 0) { bad += b.k0 != b.k1; continue; }
        bad += b.row0 != row || b.nrows > threads || b.k1 - b.k0 > COOP_EPT * threads;
        bad += b.k0 != rp[b.row0] || b.k1 != rp[b.row0 + b.nrows];
        row += b.nrows;
    }
    return bad + (row != (int64_t)rp.size() - 1);
}

}  // namespace

int main()
{
    std::mt19937 rng(71);
    int bad = 0;
    struct Case { int64_t n, m, qper, aper; int cus; };
    const Case cases[] = {
        {3000, 0, 11, 0, 256},       // no rows of A: its round has nothing to wait for
        {3000, 1, 11, 5, 256}, {3000, 1500, 11, 5, 256},   // fewer slices of A than of Q
        {1100, 9000, 5, 5, 256},     // more slices of A than of Q
        {1100, 12000, 5, 5, 32},     // more than there are CUs
        {5000, 5000, 5, 5, 256}, {9000, 4500, 11, 5, 64}, {9000, 4500, 11, 5, 40}, {1025, 3, 200, 1, 8}, {300, 200, 4, 3, 256},
    };
    for (const Case& c : cases) {
        const std::vector<int64_t> qp = rowptr(c.n, c.qper), ap = rowptr(c.m, c.aper);
        CoopLayout L;
        const bool fits = coop_layout(c.n, qp.data(), c.m, ap.data(), c.cus, L);
        if (coop_slices(c.n, qp.data(), 256).size() > (size_t)c.cus) {   // (none has over 128: slices of 256 rows)
            bad += expect("more slices than CUs refused", c.n, c.m, 0, !fits);
            continue;
        }
        bad += expect("a problem of at most one slice per CU taken", c.n, c.m, 0, fits);
        if (!fits) continue;
        const int nq = (int)L.q.size(), na = (int)L.a.size();
        bad += expect("rows of Q covered in order", c.n, c.m, L.full, covers(L.q, qp, L.threads) == 0);
        bad += expect("rows of A covered in order", c.n, c.m, L.full, covers(L.a, ap, L.threads) == 0);
        bad += expect("at most one workgroup per CU", c.n, c.m, L.full, L.full >= 1 && L.full <= c.cus);
        bad += expect("every workgroup has a slice of each", c.n, c.m, L.full, nq == L.full && na >= L.full);
        for (const int W : {1, 2, L.full - 1, L.full})
            if (W >= 1 && W <= L.full) bad += expect("rounds end", c.n, c.m, W, sound(W, nq, na, false, rng));
        // without the empty slices, or with slots apart, some workgroup waits for ever
        const int oq = (int)coop_slices(c.n, qp.data(), L.threads).size();
        const int oa = (int)coop_slices(c.m, ap.data(), L.threads).size();
        if (oq != oa && L.full > 1) {
            bad += expect("the model finds a missing post", c.n, c.m, L.full, !sound(L.full, oq, oa, false, rng));
            bad += expect("the model finds a missing post, slots apart", c.n, c.m, L.full, !sound(L.full, oq, oa, true, rng));
        }
    }
    std::printf("rounds driver: %d failure(s)\n", bad);
    return bad ? 1 : 0;
}
