// mtgp_poly.hpp -- GF(2)[x] polynomial arithmetic for jump-ahead planning.
//
// A polynomial is a bit vector in 64-bit words, bit i = coefficient of x^i.
// Host code only.  Multiplication uses the x86 carry-less multiply
// instruction; reduction modulo p uses Barrett's method with a precomputed
// quotient of x^(2d) by p (exact over GF(2)).
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <memory>
#include <mutex>
#include <vector>

namespace mtgp {
namespace poly {

using Poly = std::vector<uint64_t>;

int degree(const Poly &a);                 // -1 for the zero polynomial
void trim(Poly &a);
Poly mul(const Poly &a, const Poly &b);    // carry-less product
Poly square(const Poly &a);
Poly shl(const Poly &a, int n);            // a * x^n
Poly mod(const Poly &a, const Poly &p);    // schoolbook remainder
Poly divq(const Poly &a, const Poly &p);   // schoolbook quotient
Poly gcd(Poly a, Poly b);
Poly lcm(const Poly &a, const Poly &b);

// Reducer for one modulus p of degree d >= 1.
struct Modulus {
    Poly p;
    int d = 0;
    Poly mu;  // floor(x^(2d) / p)
    explicit Modulus(const Poly &p_);
    Poly reduce(const Poly &a) const;  // a mod p (Barrett when deg(a) < 2d)
    Poly mulmod(const Poly &a, const Poly &b) const;
    Poly sqrmod(const Poly &a) const;
    Poly powx(uint64_t e) const;        // x^e mod p
};

// Berlekamp-Massey on n bits (one per byte).  Returns L and the
// annihilating polynomial P(x) = x^L C(1/x) of the sequence, i.e.
// sum_i P_i s_{t+i} = 0 for all t with t+L < n.
int berlekamp_massey(const uint8_t *bits, int n, Poly *annihilator);

// The first nbits coefficients, 32 per word.
std::vector<uint32_t> pack32(const Poly &p, int nbits);

// g[c-1] = x^(c*lseg-1) mod p for c = 1 .. g.size(), packed to deg p bits.
struct PowerSet {
    uint64_t lseg = 0;
    std::vector<std::vector<uint32_t>> g;
};

// One modulus's power sets.  A set costs a modular product per power, far
// more than a batch that uses it, so sets of other segment lengths are kept
// beside the one in use: requests of many lengths, or small batches between
// large ones, then do not build them again and again.  The others together
// are kept to max(POWERS_KEEP_BYTES, the used set's size), least recently
// used first to go.  Safe with several threads; a set that was handed out
// never changes.
constexpr size_t POWERS_KEEP_BYTES = 64 << 10;
class Powers {
   public:
    // The set of this length with at least n powers, or null.
    std::shared_ptr<const PowerSet> find(uint64_t lseg, int n);
    // The same, built or extended if need be.
    std::shared_ptr<const PowerSet> get(const Modulus &m, uint64_t lseg, int n);
    size_t built() const;   // powers computed so far
    size_t bytes() const;   // of the sets held

   private:
    std::shared_ptr<PowerSet> front(uint64_t lseg);  // the set, moved to the front, or null
    mutable std::mutex mu_;
    std::vector<std::shared_ptr<PowerSet>> sets_;    // most recently used first
    size_t built_ = 0;
};

}  // namespace poly
}  // namespace mtgp
