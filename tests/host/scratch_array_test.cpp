// Host-only check of the growing scratch arrays: a stand-in for the GPU runtime fails on demand and counts what is allocated.
// Prints one line per expectation; exit status 0 when every one holds.
#include "scratch_array.hpp"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>

namespace {
std::set<void *> g_live;
int g_fail_allocate = 0, g_fail_zero = 0, g_strangers = 0;      // calls until one fails; releases of what was not allocated

struct MockApi {
    static bool synchronize() { return true; }
    static bool allocate(void **out, size_t n) {
        if (g_fail_allocate && --g_fail_allocate == 0) return false;
        *out = std::malloc(n);
        std::memset(*out, 0xAB, n);
        g_live.insert(*out);
        return true;
    }
    static bool release(void *p) {
        if (!g_live.erase(p)) { ++g_strangers; return false; }
        std::free(p);
        return true;
    }
    static bool zero(void *p, size_t n) {
        if (g_fail_zero && --g_fail_zero == 0) return false;
        std::memset(p, 0, n);
        return true;
    }
    static void clear_error() {}
};
typedef srs::BasicScratchArray<MockApi, uint32_t> Array;

int check(const char *what, bool cond) {
    std::printf("%s: %s\n", what, cond ? "ok" : "FAILED");
    return cond ? 0 : 1;
}
bool zeros(const Array &a) {
    for (uint64_t k = 0; k < a.cap; ++k)
        if (a.p[k]) return false;
    return true;
}
}  // namespace

int main() {
    int bad = 0;
    uint32_t piece[64];
    std::memset(piece, 0, sizeof(piece));
    for (int fault = 0; fault < 3; ++fault) {              // none, the allocation, the zeroing
        Array a;
        a.begin(piece, 64);
        bad += check("what fits stays where it is", a.grow(64) && a.p == piece && g_live.empty());
        bad += check("grows", a.grow(100) && a.p != piece && a.cap == 100 && zeros(a) && g_live.size() == 1);
        piece[3] = 7;                                      // left there by earlier calls
        g_fail_allocate = fault == 1; g_fail_zero = fault == 2 ? 2 : 0;
        const bool grew = a.grow(200);
        bad += check("a failure is reported", grew == (fault == 0));
        if (!grew) {
            bad += check("and leaves the piece it began as", a.p == piece && a.cap == 64 && zeros(a) && g_live.empty());
            bad += check("what fits the piece is served from it", a.grow(10) && a.p == piece && g_live.empty());
            bad += check("a larger request tries again", a.grow(70) && a.p != piece && a.cap == 70 && zeros(a) && g_live.size() == 1);
        }
        a.release();
        bad += check("nothing is left, nothing foreign released", g_live.empty() && g_strangers == 0 && a.p == piece);
    }
    return bad ? 1 : 0;
}
