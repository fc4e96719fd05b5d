// Host checks where no thread, or no memory for one, is to be had: the parts
// that the threads would take are looked at by the caller, and nothing leaves
// the C entry but its status. Built with g++ by tests/test_host_threads.py.
#include <cerrno>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <pthread.h>
#include <vector>

#include "mincut.h"

static bool no_thread = false;
static bool no_memory = false;

extern "C" int pthread_create(pthread_t*, const pthread_attr_t*, void* (*)(void*), void*) {
    if (!no_thread) std::abort();   // the other case ends before a thread is asked for
    return EAGAIN;
}
void* operator new(size_t bytes) {
    if (no_memory) throw std::bad_alloc();
    if (void* p = std::malloc(bytes)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

int main() {
    const int32_t n = 1000, nnz = 1 << 21;   // several parts
    std::vector<int32_t> rp(n + 1), col(nnz);
    std::vector<int64_t> w(nnz, 1);
    for (int32_t v = 0; v <= n; v++) rp[v] = (int32_t)((int64_t)nnz * v / n);
    for (int32_t j = 0; j < nnz; j++) col[j] = j % n;
    const mc_csr g{n, nnz, rp.data(), col.data(), w.data(), MC_HOST};
    for (int kind = 0; kind < 2; kind++) {
        (kind ? no_memory : no_thread) = true;
        const mc_status ok = mc_check_graph(&g, 0);
        no_memory = no_thread = false;
        if (ok != MC_OK) return std::printf("kind %d: status %d\n", kind, ok), 1;
        std::printf("kind %d ok\n", kind);
        std::fflush(stdout);
    }
    return 0;
}
