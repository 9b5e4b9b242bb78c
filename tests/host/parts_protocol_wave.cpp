// The protocol of parts_protocol.cpp in the finer steps of the kernel whose halo words are copied by a
// wave of their own: within a step of a workgroup the updates of single sites (each publishing
// its boundary word) and the copies of single halo words for the coming step run in any order
// and end at a barrier, while the other workgroup stands anywhere in its own steps.  So a copy may
// come before or between the updates of its step, and a workgroup may see part of a plane
// published.  Where the last wave does both (no wave left for the halo) its own sites come
// first.  Results against the unsplit sweeps bit for bit, no interleaving may leave both
// workgroups waiting, and a launch after one whose waits timed out agrees too.  A copy into the
// slots that the same step reads (planted here) has to be seen.
#define main parts_protocol_main
#include "parts_protocol.cpp"
#undef main

struct Wave {
    int p, w = 0, pi = 0;
    std::vector<double> xl;
    std::vector<int> sites, words;  // of this step, not yet done
    int own = 0;                    // updates that the copying wave has to do first (they lead `sites`)
    bool final_copy = false, done = false, gave_up = false;
};

enum Mode { OWN_WAVE, SHARED_WAVE, PLANTED };

static int launch_wave(const Problem &Q, const std::vector<double> &v, unsigned epoch, std::vector<Word> &xch, int stall_part,
                       Mode mode, bool skip_turns, std::mt19937 &rng, std::vector<double> &xs, bool *timed_out, std::string &msg) {
    const HostTables &T = Q.T;
    const PartTables &P = Q.P;
    const int Vp = P.Vp, Hp = P.Hp, H = T.nplanes, nsw = 2 * Q.n_ssor;
    auto word = [&](int q, int sweep, int k) -> Word & { return xch[((size_t)q * 3 + sweep % 3) * Hp + k]; };
    auto plane = [&](const Wave &A) { return (A.w & 1) == 0 ? A.pi : H - 1 - A.pi; };
    auto version = [&](const Wave &A) { return ((A.p == 0) == ((A.w & 1) == 0)) ? A.w : A.w - 1; };
    auto begin = [&](Wave &A) {
        const int h = plane(A), *st = &P.imp_start[(size_t)A.p * (MAX_PLANES + 1)];
        A.sites.clear();
        A.words.clear();
        for (int i = P.pstart[h]; i < P.pstart[h + 1]; ++i) A.sites.push_back(i);
        A.own = mode == SHARED_WAVE ? (int)A.sites.size() / 8 : 0;
        if (A.pi + 1 < H && version(A) >= 0) {
            const int hn = mode == PLANTED ? h : (A.w & 1) == 0 ? h + 1 : h - 1;
            for (int e = st[hn]; e < st[hn + 1]; ++e) A.words.push_back(P.imp[(size_t)A.p * Hp + e]);
        }
    };
    Wave parts[2];
    for (int p = 0; p < 2; ++p) {
        parts[p].p = p;
        parts[p].xl.assign(Vp + Hp + 1, 0.0);
        begin(parts[p]);
    }
    auto take = [&](std::vector<int> &l, size_t j) {
        const int e = l[j];
        l[j] = l.back();
        l.pop_back();
        return e;
    };
    auto update_site = [&](Wave &A, int i) {
        const int s = P.gslot[(size_t)A.p * Vp + i];
        if (!(skip_turns && A.w > 0 && A.pi == 0))
            A.xl[i] = update(Q, v, s, [&](int k) {
                const int mu = k >> 1, d = k & 1;
                const unsigned wd = P.pnb[(((size_t)A.p * Vp + i) * 2 + d) * 2 + (mu >> 1)];
                return A.xl.at((mu & 1) ? wd >> 16 : wd & 0xffffu);
            });
        const int kx = P.exp_idx[(size_t)A.p * Vp + i];
        if (kx >= 0) word(A.p, A.w, kx) = Word{A.xl[i], tagof(epoch, A.w)};
    };
    // one action; false when every one that is left waits for a word
    auto advance = [&](Wave &A) -> bool {
        if (A.sites.empty() && A.words.empty()) {  // the barrier
            if (A.final_copy) { A.done = true; return true; }
            if (++A.pi == H) {
                A.pi = 0;
                if (++A.w == nsw) {
                    A.final_copy = true;
                    for (int k = 0; k < Hp; ++k) A.words.push_back(k);
                    return true;
                }
            }
            begin(A);
            return true;
        }
        const int ver = A.final_copy ? nsw - 1 : version(A);
        const size_t n = A.sites.size() + A.words.size(), at = rng() % n;
        for (size_t r = 0; r < n; ++r) {
            const size_t j = (at + r) % n;
            if (j < A.sites.size()) {
                // the leading `own` ones by the copying wave, the rest by the others, in any order
                if ((int)j < A.own) --A.own, std::swap(A.sites[j], A.sites[A.own]), update_site(A, take(A.sites, A.own));
                else update_site(A, take(A.sites, j));
                return true;
            }
            if (A.own > 0) continue;
            const size_t m = j - A.sites.size();
            const Word &x = word(A.p ^ 1, ver, A.words[m]);
            if (x.tag != tagof(epoch, ver) && !A.gave_up) continue;
            A.xl[Vp + A.words[m]] = x.v;
            take(A.words, m);
            return true;
        }
        return false;
    };
    *timed_out = false;
    while (!parts[0].done || !parts[1].done) {
        const int first = (int)(rng() & 1u);
        const int burst = (rng() % 4 == 0) ? 1 + (int)(rng() % 3000) : 1 + (int)(rng() % 40);
        bool moved = false;
        for (int t = 0; t < 2 && !moved; ++t) {
            Wave &A = parts[(first + t) & 1];
            if (A.p == stall_part && !parts[A.p ^ 1].gave_up) continue;
            for (int r = 0; r < burst && !A.done && advance(A); ++r) moved = true;
        }
        if (!moved) {
            Wave *W = nullptr;
            for (auto &A : parts)
                if (!A.done && !A.gave_up && stall_part >= 0) W = &A;
            if (W && W->p == stall_part && !parts[W->p ^ 1].done && !parts[W->p ^ 1].gave_up) W = &parts[W->p ^ 1];
            if (!W) { msg = "both workgroups wait: deadlock"; return 1; }
            W->gave_up = *timed_out = true;
        }
    }
    xs.assign(T.Vb, 0.0);
    for (int p = 0; p < 2; ++p)
        for (int i = 0; i < Vp; ++i) xs[P.gslot[(size_t)p * Vp + i]] = parts[p].xl[i];
    return 0;
}

static int run_wave(const int B[4], const int S[4], int n_ssor, unsigned seed, Mode mode, bool skip_turns, bool fail_first, std::string &msg) {
    Problem Q;
    if (!make_problem(B, S, n_ssor, seed, Q, msg)) return 2;
    std::vector<Word> xch((size_t)2 * 3 * Q.P.Hp, Word{0.0, 0u});
    std::mt19937 rng(seed);
    std::vector<double> xs;
    bool to = false;
    unsigned epoch = 1u;
    if (fail_first) {
        if (launch_wave(Q, source(Q.T.Vb, seed + 2000), epoch, xch, (int)(seed & 1u), mode, skip_turns, rng, xs, &to, msg)) return 1;
        if (!to) { msg = "the slow part did not make a wait time out"; return 1; }
        const unsigned after[4] = {0u, 0u, epoch + 1u, 1u};
        unsigned next[4];
        parts_sync_after_error(after, next);
        epoch = next[2];
    }
    const std::vector<double> v = source(Q.T.Vb, seed + 1000);
    if (launch_wave(Q, v, epoch, xch, -1, mode, skip_turns, rng, xs, &to, msg)) return 1;
    if (to) { msg = "a wait timed out in a launch without a slow part"; return 1; }
    return compare(xs, whole_block(Q, v), msg);
}

int main() {
    struct Case { int B[4], S[4], n_ssor; } cases[] = {
        {{6, 6, 6, 12}, {3, 3, 3, 6}, 4}, {{4, 4, 4, 4}, {2, 2, 2, 2}, 4},  {{4, 4, 4, 8}, {2, 2, 2, 2}, 3},
        {{6, 6, 6, 6}, {3, 3, 3, 3}, 2},  {{4, 6, 4, 12}, {2, 3, 2, 3}, 4}, {{8, 8, 6, 6}, {2, 2, 3, 3}, 2}};
    int fails = 0, seen = 0;
    for (auto &cs : cases)
        for (unsigned seed = 1; seed <= 12; ++seed) {
            std::string msg;
            const Mode mode = seed % 2 ? OWN_WAVE : SHARED_WAVE;
            if (run_wave(cs.B, cs.S, cs.n_ssor, seed, mode, seed > 6, seed % 3 == 0, msg)) {
                printf("FAIL B=%dx%dx%dx%d S=%dx%dx%dx%d n_ssor=%d seed=%u: %s\n", cs.B[0], cs.B[1], cs.B[2], cs.B[3], cs.S[0], cs.S[1],
                       cs.S[2], cs.S[3], cs.n_ssor, seed, msg.c_str());
                ++fails;
            }
            std::string m2;
            if (seed <= 3 && run_wave(cs.B, cs.S, cs.n_ssor, seed, PLANTED, false, false, m2)) ++seen;
        }
    printf("copies into the slots of their own step: seen in %d of %d cases\n", seen, (int)(sizeof cases / sizeof cases[0]) * 3);
    if (seen == 0) ++fails;
    printf(fails ? "%d failures\n" : "all protocol cases agree\n", fails);
    return fails ? 1 : 0;
}
