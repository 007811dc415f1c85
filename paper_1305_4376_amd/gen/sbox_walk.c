/*
 * sbox_walk.c -- makes a circuit of 3-input lookup gates for one S-box smaller
 * by a random walk over correct circuits.
 *
 * Build-time tool.  Input: the S-box's 64 entries (argument list) and a correct
 * circuit (stdin, the format that sbox_search.c prints).  Output (stdout): the
 * start and every smaller circuit as it is found; the last block is the best.
 *
 * Functions are truth tables over the 64 input points, as in sbox_search.c.
 * The walk needs no cost function besides the size: what a gate has to compute
 * matters only at the points where its value reaches an output (the care set,
 * found by flipping the gate and evaluating what follows), so most gates can
 * be rebuilt in many ways, and a step takes one of them at random.
 *   rewire   one gate becomes another node where an existing one (or its
 *            complement) agrees on the care set, which saves a gate; else a
 *            random gate over three nodes that do not depend on it, drawn from
 *            those that agree on the care set.
 *   rebuild  one gate, with all gates that only it uses, becomes two gates
 *            F(G(a, b, c), d, e) for a random pair (d, e): G must equal the
 *            target or its complement on every cell of (d, e) where the target
 *            is not constant, a parity problem over four cells.
 * Gates that no output needs any more are dropped: that is where the size
 * falls.  A step never leaves the correct circuits; it is taken back if it makes the
 * circuit larger than the smallest so far by more than SLACK gates.
 */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef uint64_t tt;

#define MAXN 80

typedef struct {
    int in[3];
    int lut; /* bit 4a + 2b + c */
} gate_t;

typedef struct {
    int n; /* nodes 0..5 are inputs; operands come before their gate */
    gate_t g[MAXN];
    tt v[MAXN];
    int out[4];
} circuit_t;

static tt target[4];
static uint64_t rng_state = 0x9E3779B97F4A7C15ull;

static uint64_t rnd(void) {
    uint64_t z = (rng_state += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
static int rndint(int n) { return (int)((rnd() >> 33) % (uint64_t)n); }

static tt input_tt(int i) {
    tt v = 0;
    for (int p = 0; p < 64; p++)
        if ((p >> (5 - i)) & 1) v |= 1ull << p;
    return v;
}

static tt lut2(int q, tt b, tt c) {
    return (q & 1 ? ~b & ~c : 0) | (q & 2 ? ~b & c : 0) | (q & 4 ? b & ~c : 0) | (q & 8 ? b & c : 0);
}
static tt lut3(int lut, tt a, tt b, tt c) { return (~a & lut2(lut & 15, b, c)) | (a & lut2(lut >> 4, b, c)); }
static tt gate_value(const gate_t *g, const tt *v) { return lut3(g->lut, v[g->in[0]], v[g->in[1]], v[g->in[2]]); }
static tt cell3(int m, tt a, tt b, tt c) { return (m & 4 ? a : ~a) & (m & 2 ? b : ~b) & (m & 1 ? c : ~c); }

static void evaluate(circuit_t *C) {
    for (int k = 6; k < C->n; k++) C->v[k] = gate_value(&C->g[k], C->v);
}

static int correct(const circuit_t *C) {
    for (int j = 0; j < 4; j++) {
        const tt x = C->v[C->out[j]] ^ target[j];
        if (x != 0 && ~x != 0) return 0;
    }
    return 1;
}

/* Appends node k of C, operands first, to D. */
static void place(const circuit_t *C, circuit_t *D, int *map, int k) {
    if (map[k] >= 0) return;
    for (int i = 0; i < 3; i++) place(C, D, map, C->g[k].in[i]);
    gate_t g = C->g[k];
    for (int i = 0; i < 3; i++) g.in[i] = map[g.in[i]];
    map[k] = D->n;
    D->g[D->n++] = g;
}

/* Drops operands that a gate does not depend on and gates that no output needs; restores the order. */
static void finish(circuit_t *C) {
    static const int weight[3] = {4, 2, 1};
    for (int k = 6; k < C->n; k++)
        for (int i = 0; i < 3; i++) {
            int depends = 0;
            for (int m = 0; m < 8; m++) depends |= ((C->g[k].lut >> m) ^ (C->g[k].lut >> (m ^ weight[i]))) & 1;
            if (!depends) C->g[k].in[i] = C->g[k].in[(i + 1) % 3];
        }
    int map[MAXN];
    for (int i = 0; i < MAXN; i++) map[i] = i < 6 ? i : -1;
    circuit_t D;
    D.n = 6;
    memcpy(D.v, C->v, 6 * sizeof(tt));
    for (int j = 0; j < 4; j++) place(C, &D, map, C->out[j]);
    for (int j = 0; j < 4; j++) D.out[j] = map[C->out[j]];
    evaluate(&D);
    *C = D;
}

/* after[i]: node i is k or depends on it.  Returns the points at which k's value reaches an output. */
static tt care_set(const circuit_t *C, int k, char *after) {
    tt w[MAXN];
    memcpy(w, C->v, sizeof(tt) * (size_t)C->n);
    w[k] = ~w[k];
    for (int i = 0; i <= k; i++) after[i] = i == k;
    for (int i = k + 1; i < C->n; i++) {
        const int *in = C->g[i].in;
        after[i] = after[in[0]] | after[in[1]] | after[in[2]];
        if (after[i]) w[i] = gate_value(&C->g[i], w);
    }
    tt care = 0;
    for (int j = 0; j < 4; j++) care |= w[C->out[j]] ^ C->v[C->out[j]];
    return care;
}

/* Can a gate over a, b, c be 1 on `on` and 0 on `off`? */
static int separates(tt on, tt off, tt a, tt b, tt c) {
    for (int m = 0; m < 4; m++) {
        const tt x = (m & 2 ? a : ~a) & (m & 1 ? b : ~b), p = on & x, q = off & x;
        if (p && q && (((p & c) && (q & c)) || ((p & ~c) && (q & ~c)))) return 0;
    }
    return 1;
}

/* A filter for separates: 64 pairs of a point of `on` and a point of `off` drawn at random, every pair inside one
   of the cells given; apart[i]: the pairs that candidate i tells apart.  A gate can only separate if its three
   operands tell all pairs apart between them.  Returns 0 if no cell has both kinds of points. */
static int sample_pairs(const circuit_t *C, const int *cand, int n, const tt *on, const tt *off, int cells, uint64_t *apart) {
    int point[2][64], count[2] = {0, 0}, mixed[4], n_mixed = 0, p[64], q[64];
    for (int m = 0; m < cells; m++)
        if (on[m] && off[m]) mixed[n_mixed++] = m;
    if (n_mixed == 0) return 0;
    for (int t = 0; t < 64; t++) {
        if (t % (64 / n_mixed) == 0 && t / (64 / n_mixed) < n_mixed) {
            const int m = mixed[t / (64 / n_mixed)];
            count[0] = count[1] = 0;
            for (tt x = on[m]; x; x &= x - 1) point[0][count[0]++] = __builtin_ctzll(x);
            for (tt x = off[m]; x; x &= x - 1) point[1][count[1]++] = __builtin_ctzll(x);
        }
        const uint64_t r = rnd();
        p[t] = point[0][(r & 0xffffffff) % (unsigned)count[0]];
        q[t] = point[1][(r >> 32) % (unsigned)count[1]];
    }
    for (int i = 0; i < n; i++) {
        const tt v = C->v[cand[i]];
        uint64_t a = 0;
        for (int t = 0; t < 64; t++) a |= ((v >> p[t] ^ v >> q[t]) & 1) << t;
        apart[i] = a;
    }
    return 1;
}

/* Such a gate; cells without a requirement at random. */
static gate_t make_gate(const circuit_t *C, tt on, tt off, int a, int b, int c) {
    gate_t g = {{a, b, c}, 0};
    for (int m = 0; m < 8; m++) {
        const tt x = cell3(m, C->v[a], C->v[b], C->v[c]);
        if ((on & x) || (!(off & x) && (rnd() >> 40 & 1))) g.lut |= 1 << m;
    }
    return g;
}

static void shuffle(int *a, int n) {
    for (int i = n - 1; i > 0; i--) {
        const int j = rndint(i + 1), t = a[i];
        a[i] = a[j];
        a[j] = t;
    }
}

/* Every use of node k becomes node r, or its complement. */
static void replace(circuit_t *C, int k, int r, int complement) {
    static const int weight[3] = {4, 2, 1};
    for (int u = 6; u < C->n; u++)
        for (int i = 0; i < 3; i++) {
            if (C->g[u].in[i] != k) continue;
            C->g[u].in[i] = r;
            if (!complement) continue;
            int lut = 0;
            for (int m = 0; m < 8; m++) lut |= ((C->g[u].lut >> (m ^ weight[i])) & 1) << m;
            C->g[u].lut = lut;
        }
    for (int j = 0; j < 4; j++)
        if (C->out[j] == k) C->out[j] = r;
}

static int rewire(circuit_t *C, int k) {
    char after[MAXN];
    const tt care = care_set(C, k, after), on = C->v[k] & care, off = ~C->v[k] & care;
    int cand[MAXN], n = 0;
    for (int i = 0; i < C->n; i++)
        if (!after[i]) cand[n++] = i;
    shuffle(cand, n);
    for (int i = 0; i < n; i++) {
        const tt x = C->v[cand[i]];
        const int same = !(on & ~x) && !(off & x), inverse = !(on & x) && !(off & ~x);
        if (!same && !inverse) continue;
        replace(C, k, cand[i], !same);
        return 1;
    }
    const int want = 1 + rndint(24); /* one of the first few in a random order */
    int found = 0, pick[3] = {0, 0, 0};
    uint64_t apart[MAXN];
    if (!sample_pairs(C, cand, n, &on, &off, 1, apart)) return 0;
    for (int a = 0; a < n && found < want; a++)
        for (int b = a + 1; b < n && found < want; b++)
            for (int c = b + 1; c < n && found < want; c++) {
                if (~(apart[a] | apart[b] | apart[c])) continue;
                if (!separates(on, off, C->v[cand[a]], C->v[cand[b]], C->v[cand[c]])) continue;
                if (rndint(++found) == 0) {
                    pick[0] = cand[a];
                    pick[1] = cand[b];
                    pick[2] = cand[c];
                }
            }
    if (found == 0) return 0;
    C->g[k] = make_gate(C, on, off, pick[0], pick[1], pick[2]);
    return 1;
}

/* The root of s and its parity to the root. */
static int root(const int *up, const int *parity, int s, int *p) {
    for (*p = 0; up[s] != s; s = up[s]) *p ^= parity[s];
    return s;
}

/* Polarity per cell under which a gate over a, b, c equals the target (on / off, per cell) or its complement. */
static int parity_gate(const tt *on, const tt *off, tt a, tt b, tt c, int *polarity) {
    int up[4] = {0, 1, 2, 3}, parity[4] = {0, 0, 0, 0};
    for (int i = 0; i < 8; i++) {
        const tt x = cell3(i, a, b, c);
        int first = -1, first_value = 0;
        for (int m = 0; m < 4; m++) {
            const int p = (on[m] & x) != 0, q = (off[m] & x) != 0;
            if (p && q) return 0;
            if (!p && !q) continue;
            if (first < 0) {
                first = m;
                first_value = p;
                continue;
            }
            int pm, pf;
            const int rm = root(up, parity, m, &pm), rf = root(up, parity, first, &pf), need = p ^ first_value;
            if (rm == rf) {
                if ((pm ^ pf) != need) return 0;
            } else {
                up[rm] = rf;
                parity[rm] = pm ^ pf ^ need;
            }
        }
    }
    for (int m = 0; m < 4; m++) root(up, parity, m, &polarity[m]);
    return 1;
}

static int rebuild(circuit_t *C, int k, int pairs, int limit) {
    char after[MAXN], cone[MAXN] = {0};
    const tt care = care_set(C, k, after), on = C->v[k] & care, off = ~C->v[k] & care;
    int cone_size = 1; /* k and the gates that only the cone uses */
    cone[k] = 1;
    for (int i = k - 1; i >= 6; i--) {
        int used = 0, inside = 1;
        for (int u = 6; u < C->n; u++)
            for (int t = 0; t < 3; t++)
                if (C->g[u].in[t] == i) {
                    used = 1;
                    inside &= cone[u];
                }
        for (int j = 0; j < 4; j++) inside &= C->out[j] != i;
        if (used && inside) {
            cone[i] = 1;
            cone_size++;
        }
    }
    if (C->n - cone_size + 2 > limit || C->n + 1 >= MAXN) return 0;
    int cand[MAXN], n = 0;
    for (int i = 0; i < C->n; i++)
        if (!after[i] && !cone[i]) cand[n++] = i;
    shuffle(cand, n);
    for (int t = 0; t < pairs; t++) {
        const int d = cand[rndint(n)], e = cand[rndint(n)], start = rndint(n);
        if (d == e) continue;
        tt on4[4], off4[4];
        for (int m = 0; m < 4; m++) {
            const tt x = (m & 2 ? C->v[d] : ~C->v[d]) & (m & 1 ? C->v[e] : ~C->v[e]);
            const int mixed = (on & x) && (off & x);
            on4[m] = mixed ? on & x : 0;
            off4[m] = mixed ? off & x : 0;
        }
        uint64_t apart[MAXN];
        if (!sample_pairs(C, cand, n, on4, off4, 4, apart)) continue;
        for (int i = 0; i < n; i++)
            for (int a = (i + start) % n, b = 0; b < a; b++)
                for (int c = 0; c < b; c++) {
                    int pol[4];
                    if (~(apart[a] | apart[b] | apart[c])) continue;
                    if (!parity_gate(on4, off4, C->v[cand[a]], C->v[cand[b]], C->v[cand[c]], pol)) continue;
                    tt g_on = 0, g_off = 0;
                    for (int m = 0; m < 4; m++) {
                        g_on |= pol[m] ? off4[m] : on4[m];
                        g_off |= pol[m] ? on4[m] : off4[m];
                    }
                    const int g = C->n++;
                    C->g[g] = make_gate(C, g_on, g_off, cand[a], cand[b], cand[c]);
                    C->v[g] = gate_value(&C->g[g], C->v);
                    C->g[k] = make_gate(C, on, off, g, d, e);
                    return 1;
                }
    }
    return 0;
}

/* Outputs that need an instruction of their own for the XOR into the Feistel half: all but those of an
   unshared final gate with at most two operands. */
static int separate_outputs(const circuit_t *C) {
    int extra = 0;
    for (int j = 0; j < 4; j++) {
        const int o = C->out[j], *in = C->g[o].in;
        int shared = o < 6 || (in[0] != in[1] && in[0] != in[2] && in[1] != in[2]);
        for (int u = 6; u < C->n; u++)
            for (int t = 0; t < 3; t++) shared |= C->g[u].in[t] == o;
        for (int i = 0; i < j; i++) shared |= C->out[i] == o;
        extra += shared;
    }
    return extra;
}

static void print_circuit(const circuit_t *C) {
    printf("cost %d gates %d\n", C->n - 6 + separate_outputs(C), C->n - 6);
    for (int k = 6; k < C->n; k++)
        printf("g %d %d %d %d %d\n", k, C->g[k].in[0], C->g[k].in[1], C->g[k].in[2], C->g[k].lut);
    printf("out %d %d %d %d\n", C->out[0], C->out[1], C->out[2], C->out[3]);
    fflush(stdout);
}

static int read_circuit(circuit_t *C) {
    char line[160];
    int have_out = 0;
    C->n = 6;
    while (fgets(line, sizeof line, stdin)) {
        int k, a, b, c, l;
        if (sscanf(line, "g %d %d %d %d %d", &k, &a, &b, &c, &l) == 5) {
            if (k != C->n || k >= MAXN || a < 0 || a >= k || b < 0 || b >= k || c < 0 || c >= k || l < 0 || l > 255) return 0;
            C->g[C->n++] = (gate_t){{a, b, c}, l};
        } else if (sscanf(line, "out %d %d %d %d", &C->out[0], &C->out[1], &C->out[2], &C->out[3]) == 4) {
            have_out = 1;
        }
    }
    for (int j = 0; j < 4 && have_out; j++)
        if (C->out[j] < 0 || C->out[j] >= C->n) return 0;
    for (int i = 0; i < 6; i++) C->v[i] = input_tt(i);
    evaluate(C);
    return have_out && correct(C);
}

int main(int argc, char **argv) {
    if (argc < 68) {
        fprintf(stderr, "usage: sbox_walk SEED STEPS SLACK s0 .. s63 < circuit\n");
        return 2;
    }
    rng_state ^= strtoull(argv[1], NULL, 0) * 0xD1342543DE82EF95ull;
    const long steps = atol(argv[2]), kStale = 2000000;
    const int slack = atoi(argv[3]);
    for (int p = 0; p < 64; p++)
        for (int j = 0; j < 4; j++)
            if ((atoi(argv[4 + p]) >> (3 - j)) & 1) target[j] |= 1ull << p;
    circuit_t C;
    if (!read_circuit(&C)) {
        fprintf(stderr, "start circuit is not correct\n");
        return 1;
    }
    finish(&C);
    circuit_t best = C;
    int best_extra = separate_outputs(&C);
    print_circuit(&best);
    for (long step = 0, since = 0; step < steps; step++, since++) {
        circuit_t D = C;
        const int k = 6 + rndint(D.n - 6), r = rndint(100);
        /* mostly rewiring; now and then two gates in place of a cone, rarely with one gate more than before */
        if (!(r < 90 ? rewire(&D, k) : rebuild(&D, k, 6, r < 98 ? C.n : C.n + 1))) continue;
        finish(&D);
        if (!correct(&D)) {
            fprintf(stderr, "step %ld broke the circuit\n", step);
            return 1;
        }
        if (D.n > best.n + slack) continue;
        C = D;
        const int extra = separate_outputs(&C);
        if (C.n < best.n || (C.n == best.n && extra < best_extra)) {
            if (C.n < best.n) since = 0;
            best = C;
            best_extra = extra;
            print_circuit(&best);
        }
        if (since > kStale) { /* back to the best */
            since = 0;
            C = best;
        }
    }
    return 0;
}
