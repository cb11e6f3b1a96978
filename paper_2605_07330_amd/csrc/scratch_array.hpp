// A scratch array on the device that begins as a piece of a larger allocation and moves to one of its own when more is asked for.
// The runtime calls come in through a policy type, so that what happens when one fails can be tried on a machine without a GPU
// (tests/host/scratch_array_test.cpp).
//   Api::synchronize() -> bool, Api::allocate(void **, size_t) -> bool, Api::release(void *) -> bool,
//   Api::zero(void *, size_t) -> bool (done when it returns), Api::clear_error().
#pragma once

#include <cstddef>
#include <cstdint>

namespace srs {

template <class Api, class T>
struct BasicScratchArray {
    T *p = nullptr;
    uint64_t cap = 0;                       // elements
    T *built_in = nullptr;                  // the piece it began as, which belongs to somebody else
    uint64_t built_in_cap = 0;

    void begin(T *piece, uint64_t elements) { p = built_in = piece; cap = built_in_cap = elements; }

    // Room for `elements`, of which all are 0 where it moves: allocates and synchronises then.  Where that fails the array is the
    // piece it began as, zeroed, and asking again is possible.
    bool grow(uint64_t elements) {
        if (elements <= cap) return true;
        if (!Api::synchronize()) return failed();
        if (p != built_in) {
            T *const old = p;
            p = built_in; cap = built_in_cap;
            if (!Api::release(old)) return failed();
            if (built_in && !Api::zero(built_in, built_in_cap * sizeof(T))) return failed();
        }
        void *q = nullptr;
        if (!Api::allocate(&q, elements * sizeof(T))) return failed();
        if (!Api::zero(q, elements * sizeof(T))) { failed(); (void)Api::release(q); return false; }
        p = static_cast<T *>(q); cap = elements;
        return true;
    }

    void release() {
        if (p != built_in) (void)Api::release(p);
        p = built_in; cap = built_in_cap;
    }

private:
    static bool failed() { Api::clear_error(); return false; }
};

}  // namespace srs
