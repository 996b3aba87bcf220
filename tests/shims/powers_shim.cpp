// C entry points for tests/test_powers.py: one stream's cached powers.
#include <string.h>

#include "mtgp_poly.hpp"

using namespace mtgp::poly;

namespace {
struct Cache {
    Modulus m;
    Powers p;
    std::vector<std::shared_ptr<const PowerSet>> held;
    explicit Cache(const Poly &q) : m(q) {}
};
}  // namespace

extern "C" {

void *powers_new(const unsigned long long *p, int n) { return new Cache(Poly(p, p + n)); }
void powers_delete(void *c) { delete (Cache *)c; }

// 1 if the cache holds n powers of this length; built otherwise.  `out`, if
// given, receives power c (1 ..) as 32-bit words.
int powers_get(void *c, unsigned long long lseg, int n, int power, uint32_t *out) {
    Cache &k = *(Cache *)c;
    const bool there = k.p.find(lseg, n) != nullptr;
    const std::shared_ptr<const PowerSet> s = k.p.get(k.m, lseg, n);
    if (out) memcpy(out, s->g[(size_t)power - 1].data(), s->g[(size_t)power - 1].size() * 4);
    return there ? 1 : 0;
}

// Holds the set, as a plan does; held(i, power) reads it later.
void powers_hold(void *c, unsigned long long lseg, int n) {
    Cache &k = *(Cache *)c;
    k.held.push_back(k.p.get(k.m, lseg, n));
}
int powers_held(void *c, int i, int power, uint32_t *out) {
    const PowerSet &s = *((Cache *)c)->held[(size_t)i];
    memcpy(out, s.g[(size_t)power - 1].data(), s.g[(size_t)power - 1].size() * 4);
    return (int)s.g.size();
}

unsigned long long powers_built(void *c) { return ((Cache *)c)->p.built(); }
unsigned long long powers_bytes(void *c) { return ((Cache *)c)->p.bytes(); }
unsigned long long powers_keep(void) { return POWERS_KEEP_BYTES; }
}
