// host_math.cpp -- see host_math.hpp.
#include "host_math.hpp"

#include <cstring>
#include <mutex>

namespace rngx {

using u128 = unsigned __int128;

uint64_t mulmod64(uint64_t a, uint64_t b, uint64_t m) { return (uint64_t)((u128)a * b % m); }

uint64_t powmod64(uint64_t a, uint64_t e, uint64_t m)
{
    uint64_t r = 1 % m;
    a %= m;
    while (e) {
        if (e & 1) r = mulmod64(r, a, m);
        a = mulmod64(a, a, m);
        e >>= 1;
    }
    return r;
}

// Miller-Rabin with the first twelve primes as bases: deterministic for
// every n < 3.3e24, hence for all 64-bit n.
bool is_prime_u64(uint64_t n)
{
    static const uint64_t bases[] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
    if (n < 2) return false;
    for (uint64_t p : bases)
        if (n % p == 0) return n == p;
    uint64_t d = n - 1;
    int r = 0;
    while ((d & 1) == 0) { d >>= 1; ++r; }
    for (uint64_t a : bases) {
        uint64_t x = powmod64(a, d, n);
        if (x == 1 || x == n - 1) continue;
        bool composite = true;
        for (int i = 1; i < r; ++i) {
            x = mulmod64(x, x, n);
            if (x == n - 1) { composite = false; break; }
        }
        if (composite) return false;
    }
    return true;
}

static bool safe_prime_rule(uint64_t a, int log2b)
{
    uint64_t m = (a << log2b) - 1;
    return is_prime_u64(m) && is_prime_u64((m - 1) / 2);
}

const std::vector<uint16_t> &mwc16_multipliers()
{
    static std::vector<uint16_t> t = [] {
        std::vector<uint16_t> v;
        for (uint64_t a = 2; a < 65536; ++a)
            if (safe_prime_rule(a, 16)) v.push_back((uint16_t)a);
        return v;
    }();
    return t;
}

uint32_t mwc32_multiplier()
{
    static uint32_t a = [] {
        for (uint64_t c = 65535; c > 1; --c)
            if (safe_prime_rule(c, 32)) return (uint32_t)c;
        return 0u;
    }();
    return a;
}

// ---------------------------------------------------------------- GF(2)
template <int W>
Gf2Mat<W> Gf2Mat<W>::identity()
{
    Gf2Mat m;
    std::memset(m.c, 0, sizeof(m.c));
    for (int b = 0; b < 32 * W; ++b) m.c[b][b >> 5] = 1u << (b & 31);
    return m;
}

template <int W>
void Gf2Mat<W>::apply(const uint32_t *in, uint32_t *out) const
{
    uint32_t r[W] = {};
    for (int w = 0; w < W; ++w) {
        uint32_t word = in[w];
        while (word) {
            int bit = __builtin_ctz(word);
            word &= word - 1;
            const uint32_t *col = c[32 * w + bit];
            for (int i = 0; i < W; ++i) r[i] ^= col[i];
        }
    }
    std::memcpy(out, r, sizeof(r));
}

template <int W>
Gf2Mat<W> Gf2Mat<W>::operator*(const Gf2Mat &rhs) const
{
    Gf2Mat out;
    for (int b = 0; b < 32 * W; ++b) apply(rhs.c[b], out.c[b]);
    return out;
}

template <int W>
bool Gf2Mat<W>::operator==(const Gf2Mat &o) const
{
    return std::memcmp(c, o.c, sizeof(c)) == 0;
}

template struct Gf2Mat<1>;
template struct Gf2Mat<8>;

// 32x32 building blocks: I, L^k (bit i -> bit i+k), R^k (bit i -> bit i-k),
// as column arrays, composed as matrices.
using M32 = Gf2Mat<1>;

static M32 shift_mat(int k, bool left)
{
    M32 m;
    std::memset(m.c, 0, sizeof(m.c));
    for (int i = 0; i < 32; ++i) {
        int j = left ? i + k : i - k;
        if (j >= 0 && j < 32) m.c[i][0] = 1u << j;
    }
    return m;
}

static M32 add(const M32 &a, const M32 &b)
{
    M32 r;
    for (int i = 0; i < 32; ++i) r.c[i][0] = a.c[i][0] ^ b.c[i][0];
    return r;
}

static M32 I_plus_L(int k) { return add(M32::identity(), shift_mat(k, true)); }
static M32 I_plus_R(int k) { return add(M32::identity(), shift_mat(k, false)); }

// Eq. (5) as a block companion matrix on the window (v_{n-8} .. v_{n-1}):
// the new word is sum_j A_j v_{n-j}, the other words slide down by one.
Gf2Mat<8> xs256_step_matrix()
{
    M32 A[9];
    for (auto &a : A) std::memset(a.c, 0, sizeof(a.c));
    A[1] = I_plus_L(9) * I_plus_L(13);
    A[4] = I_plus_L(7);
    A[5] = I_plus_R(3);
    A[7] = I_plus_R(10);
    A[8] = I_plus_L(24) * I_plus_R(7);
    Gf2Mat<8> M;
    std::memset(M.c, 0, sizeof(M.c));
    for (int w = 0; w < 8; ++w) {       // input word w holds v_{n-8+w}
        int lag = 8 - w;
        for (int bit = 0; bit < 32; ++bit) {
            uint32_t *col = M.c[32 * w + bit];
            if (w >= 1) col[w - 1] = 1u << bit;  // slides to position w-1
            col[7] = A[lag].c[bit][0];           // contribution to v_n
        }
    }
    return M;
}

// Eq. (6), applied as written: first (I+L^13), then (I+R^17), then (I+L^5).
Gf2Mat<1> xs32_step_matrix() { return I_plus_L(5) * I_plus_R(17) * I_plus_L(13); }

// ---------------------------------------------------------------- tables
// Polynomials over GF(2) of degree below 256, bit i the coefficient of x^i.
struct Gf2Poly {
    uint64_t w[4];
};

// x a mod (x^256 + f).
static Gf2Poly poly_mulx(Gf2Poly a, const Gf2Poly &f)
{
    const uint64_t top = 0 - (a.w[3] >> 63);
    for (int k = 3; k > 0; --k) a.w[k] = (a.w[k] << 1) | (a.w[k - 1] >> 63);
    a.w[0] <<= 1;
    for (int k = 0; k < 4; ++k) a.w[k] ^= f.w[k] & top;
    return a;
}

// The 16 products of a by the polynomials of degree below 4.
static void poly_nibbles(const Gf2Poly &a, const Gf2Poly &f, Gf2Poly (&t)[16])
{
    t[0] = Gf2Poly{{0, 0, 0, 0}};
    t[1] = a;
    for (int v = 2; v < 16; v *= 2) {
        t[v] = poly_mulx(t[v / 2], f);
        for (int u = 1; u < v; ++u)
            for (int k = 0; k < 4; ++k) t[v + u].w[k] = t[v].w[k] ^ t[u].w[k];
    }
}

// a b mod (x^256 + f), four bits of b at a time.
static Gf2Poly poly_mulmod(const Gf2Poly &a, const Gf2Poly &b, const Gf2Poly &f)
{
    Gf2Poly ta[16], tf[16], r{{0, 0, 0, 0}};
    poly_nibbles(a, f, ta);
    poly_nibbles(f, f, tf);  // v x^256
    for (int i = 63; i >= 0; --i) {
        const Gf2Poly &over = tf[r.w[3] >> 60], &add = ta[(b.w[i / 16] >> (4 * (i % 16))) & 15];
        for (int k = 3; k > 0; --k) r.w[k] = (r.w[k] << 4) | (r.w[k - 1] >> 60);
        r.w[0] <<= 4;
        for (int k = 0; k < 4; ++k) r.w[k] ^= over.w[k] ^ add.w[k];
    }
    return r;
}

// The characteristic polynomial x^256 + f of the XS256 step, as the shortest
// recurrence of one bit of its output (Berlekamp-Massey, Massey 1969); the step
// has the full period, so the recurrence has degree 256.
static Gf2Poly xs256_char_poly()
{
    constexpr int n = 640;
    const Gf2Mat<8> M = xs256_step_matrix();
    std::vector<int> bit(n);
    uint32_t v[8] = {1, 0, 0, 0, 0, 0, 0, 0}, u[8];
    for (int i = 0; i < n; ++i) {
        M.apply(v, u);
        std::memcpy(v, u, sizeof(v));
        bit[i] = v[7] & 1;
    }
    std::vector<int> C(n + 1), B(n + 1), t;
    C[0] = B[0] = 1;
    int L = 0, m = 1;
    for (int i = 0; i < n; ++i, ++m) {
        int d = bit[i];
        for (int k = 1; k <= L; ++k) d ^= C[k] & bit[i - k];
        if (!d) continue;
        t = C;
        for (int k = 0; k + m <= n; ++k) C[k + m] ^= B[k];
        if (2 * L <= i) {
            L = i + 1 - L;
            B = t;
            m = 0;
        }
    }
    Gf2Poly f{{0, 0, 0, 0}};  // x^256 C(1/x)
    for (int k = 1; k <= 256; ++k)
        if (C[k]) f.w[(256 - k) / 64] |= (uint64_t)1 << ((256 - k) % 64);
    return f;
}

static HostTables *build_tables()
{
    auto *T = new HostTables();
    T->mwc32_a = mwc32_multiplier();
    T->mwc32_m = ((uint64_t)T->mwc32_a << 32) - 1;
    const auto &t = mwc16_multipliers();
    for (int i = 0; i < kMwc16Count; ++i) T->t392[i] = t[i];

    const uint64_t m = T->mwc32_m;
    const uint64_t two64 = mulmod64(((uint64_t)1 << 32) % m, ((uint64_t)1 << 32) % m, m);
    uint64_t p = T->mwc32_a;  // a^(2^0)
    for (int b = 0; b < kPowBits; ++b) {
        T->mwc32_pow_fold[b] = mulmod64(p, two64, m);
        p = mulmod64(p, p, m);
    }

    uint32_t A = 69069u, C = 1234567u;  // eq. (7)
    for (int b = 0; b < kPowBits; ++b) {
        T->lcg_pow[b][0] = A;
        T->lcg_pow[b][1] = C;
        C = A * C + C;  // (A,C) o (A,C)
        A = A * A;
    }

    M32 x = xs32_step_matrix();
    for (int b = 0; b < kPowBits; ++b) {
        for (int i = 0; i < 32; ++i) T->xs32_pow[b][i] = x.c[i][0];
        x = x * x;
    }

    for (int i = 0; i < kMwc16Count; ++i) {
        uint64_t a = t[i], mi = (a << 16) - 1;
        uint64_t two48 = powmod64(2, 48, mi);
        uint64_t q = a;
        for (int b = 0; b < kPowBits; ++b) {
            T->mwc16_pow_fold[i][b] = (uint32_t)mulmod64(q, two48, mi);
            q = mulmod64(q, q, mi);
        }
    }

    T->xs256_pow.resize((size_t)kPowBits * 256 * 8);
    auto *M = new Gf2Mat<8>(xs256_step_matrix());
    for (int b = 0; b < kPowBits; ++b) {
        std::memcpy(&T->xs256_pow[(size_t)b * 2048], M->c, sizeof(M->c));
        *M = (*M) * (*M);
    }
    delete M;
    // One table per hexadecimal digit d != 0 at position j: a jump by k then
    // takes one product per nonzero digit of k instead of one per set bit.
    T->xs256_t4w.resize((size_t)16 * 15 * 8192);
    auto *base = new Gf2Mat<8>, *P = new Gf2Mat<8>;
    for (int j = 0; j < 16; ++j) {
        std::memcpy(base->c, &T->xs256_pow[(size_t)(4 * j) * 2048], sizeof(base->c));
        *P = *base;
        for (int d = 1; d <= 15; ++d) {
            if (d > 1) *P = (*P) * (*base);
            xs256_nibble_table(&P->c[0][0], &T->xs256_t4w[((size_t)j * 15 + (d - 1)) * 8192]);
        }
    }
    delete base;
    delete P;
    const Gf2Poly f = xs256_char_poly();
    Gf2Poly xp{{2, 0, 0, 0}};  // x^(2^j)
    T->xs256_poly.resize((size_t)8 * 64 * 8);
    for (int j = 0; j <= 12; ++j) {
        if (j >= 5) {
            Gf2Poly c{{1, 0, 0, 0}};
            for (int l = 0; l < 64; ++l) {
                std::memcpy(&T->xs256_poly[((size_t)(j - 5) * 64 + l) * 8], c.w, sizeof(c.w));
                c = poly_mulmod(c, xp, f);
            }
        }
        xp = poly_mulmod(xp, xp, f);
    }
    std::memcpy(T->xs256_char, f.w, sizeof(f.w));
    T->xs256_digit.resize((size_t)16 * 15 * 8);
    xp = Gf2Poly{{2, 0, 0, 0}};  // x^(16^j)
    for (int j = 0; j < 16; ++j) {
        Gf2Poly c{{1, 0, 0, 0}};
        for (int d = 1; d <= 15; ++d) {
            c = poly_mulmod(c, xp, f);
            std::memcpy(&T->xs256_digit[((size_t)j * 15 + (d - 1)) * 8], c.w, sizeof(c.w));
        }
        xp = poly_mulmod(c, xp, f);
    }
    return T;
}

void xs256_nibble_table(const uint32_t *cols, uint32_t *t4)
{
    for (int p = 0; p < 64; ++p)
        for (int h = 0; h < 2; ++h)
            for (int v = 0; v < 16; ++v)
                for (int w = 0; w < 4; ++w) {
                    uint32_t x = 0;
                    for (int k = 0; k < 4; ++k)
                        if ((v >> k) & 1) x ^= cols[(4 * p + k) * 8 + 4 * h + w];
                    t4[((p * 2 + h) * 16 + v) * 4 + w] = x;
                }
}

const HostTables &host_tables()
{
    static HostTables *T = build_tables();
    return *T;
}

void xs256_jump_poly(uint64_t k, uint32_t poly[8])
{
    const HostTables &T = host_tables();
    Gf2Poly f, c{{1, 0, 0, 0}}, x;
    std::memcpy(f.w, T.xs256_char, sizeof(f.w));
    bool first = true;
    for (int j = 0; j < 16; ++j) {
        const int d = (int)(k >> (4 * j)) & 15;
        if (!d) continue;
        std::memcpy(x.w, &T.xs256_digit[((size_t)j * 15 + (d - 1)) * 8], sizeof(x.w));
        c = first ? x : poly_mulmod(c, x, f);
        first = false;
    }
    std::memcpy(poly, c.w, sizeof(c.w));
}

uint64_t mwc32_fold_const(uint64_t k)
{
    const HostTables &T = host_tables();
    const uint64_t m = T.mwc32_m;
    const uint64_t two64 = mulmod64(((uint64_t)1 << 32) % m, ((uint64_t)1 << 32) % m, m);
    return mulmod64(powmod64(T.mwc32_a, k, m), two64, m);
}

void xs32_lcg_jump(uint64_t k, uint32_t cols[32], uint32_t *lcg_a, uint32_t *lcg_c)
{
    const HostTables &T = host_tables();
    uint32_t A = 1, C = 0;  // identity affine map
    for (int i = 0; i < 32; ++i) cols[i] = 1u << i;
    for (int b = 0; b < kPowBits; ++b) {
        if (!((k >> b) & 1)) continue;
        const uint32_t pa = T.lcg_pow[b][0], pc = T.lcg_pow[b][1];
        C = pa * C + pc;  // 2^b more steps after the current map
        A = pa * A;
        // column i <- M^(2^b) column i, branch-free with the columns innermost
        // (data-dependent branches here cost more than the arithmetic)
        uint32_t next[32] = {0};
        for (int j = 0; j < 32; ++j) {
            const uint32_t pj = T.xs32_pow[b][j];
            for (int i = 0; i < 32; ++i) next[i] ^= pj & (0u - ((cols[i] >> j) & 1u));
        }
        for (int i = 0; i < 32; ++i) cols[i] = next[i];
    }
    *lcg_a = A;
    *lcg_c = C;
}

}  // namespace rngx
