// The store of host memory blocks on counted memory: what it keeps, what it hands out and when it allocates.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <map>
#include <thread>
#include <vector>

#include "../paper_1804_06609_amd/csrc/host_blocks.hpp"

using namespace dba;

static std::mutex g_lock;
static std::map<void *, size_t> g_held;       // allocated and not released
static size_t g_allocs, g_releases, g_bytes;
static bool g_none;

struct Counted {
    static void *allocate(size_t n)
    {
        std::lock_guard<std::mutex> hold(g_lock);
        if (g_none) return nullptr;
        void *p = malloc(n);
        g_held[p] = n;
        ++g_allocs;
        g_bytes += n;
        return p;
    }
    static void release(void *p)
    {
        std::lock_guard<std::mutex> hold(g_lock);
        if (!g_held.count(p)) { printf("released twice\n"); exit(1); }
        g_bytes -= g_held[p];
        g_held.erase(p);
        ++g_releases;
        free(p);
    }
};
typedef HostBlocks<Counted> Store;

#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); exit(1); } } while (0)

int main()
{
    const size_t K = 1024, M = 1024 * 1024;
    {
        // two large users gone, then many small ones: nothing to allocate, nothing to free
        static Store s;
        HostBlock a = s.get(M), b = s.get(900 * K);
        CHECK(a.bytes == M && b.bytes == M);
        s.put(a); s.put(b);
        const size_t allocs = g_allocs, releases = g_releases;
        for (int i = 0; i < 50; ++i) {
            HostBlock c = s.get(10 * K);
            CHECK(c.p && c.bytes >= 10 * K);
            s.put(c);
        }
        CHECK(g_allocs == allocs && g_releases == releases);
        // two at a time: one more block, one free at most, then none
        for (int i = 0; i < 50; ++i) {
            HostBlock c = s.get(10 * K), d = s.get(10 * K), e = s.get(10 * K);
            s.put(c); s.put(d); s.put(e);
        }
        CHECK(g_allocs <= allocs + 3 && g_releases <= releases + 2);
    }
    {
        // small ones kept, then large users: the small ones go, not the large blocks again and again
        static Store s;
        std::vector<HostBlock> v;
        for (int i = 0; i < 40; ++i) v.push_back(s.get(64 * K));
        for (auto &x : v) s.put(x);
        const size_t allocs = g_allocs;
        for (int i = 0; i < 50; ++i) {
            HostBlock a = s.get(M), b = s.get(M);
            s.put(a); s.put(b);
        }
        CHECK(g_allocs == allocs + 2);
    }
    {
        // several threads: never more kept than meant, no block with two users, none too small
        static Store s;
        const size_t before = g_bytes;
        std::vector<std::thread> threads;
        for (unsigned t = 0; t < 4; ++t)
            threads.emplace_back([t] {
                unsigned r = 77 + t;
                auto next = [&r] { return (r = r * 1664525u + 1013904223u) >> 8; };
                std::vector<HostBlock> mine;
                for (int i = 0; i < 20000; ++i) {
                    if (mine.size() < 6 && next() % 2) {
                        const size_t n = 1 + next() % (M + M / 8);
                        HostBlock b = s.get(n);
                        CHECK(n > M ? !b.p : (b.p && b.bytes >= n));
                        if (!b.p) continue;
                        *reinterpret_cast<volatile uint32_t *>(b.p) = t;
                        mine.push_back(b);
                    } else if (!mine.empty()) {
                        CHECK(*reinterpret_cast<volatile uint32_t *>(mine.back().p) == t);
                        s.put(mine.back());
                        mine.pop_back();
                    }
                }
                for (auto &b : mine) s.put(b);
            });
        for (auto &th : threads) th.join();
        CHECK(g_bytes - before <= Store::kKeepBytes);
    }
    {
        static Store s;
        g_none = true;
        HostBlock a = s.get(5);
        CHECK(!a.p && a.bytes == 0);
        s.put(a);
        g_none = false;
    }
    printf("host_blocks_driver ok\n");
    return 0;
}
