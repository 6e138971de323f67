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
        // blocks that somebody still writes to: nothing waits for them, they are not handed out before their words have come, and then are
        static Store s;
        std::vector<HostBlock> v;
        for (int i = 0; i < 50; ++i) {
            v.push_back(s.get(64 * K));
            for (uint32_t j = 0; j < 33; ++j) reinterpret_cast<uint32_t *>(v[i].p)[j] = 7 << 2 | j % 4;
        }
        for (auto &x : v) s.put_when(x, 33, 8 << 2, ~3u);
        auto in_v = [&](HostBlock b) {
            for (auto &x : v)
                if (x.p == b.p) return true;
            return false;
        };
        HostBlock other = s.get(64 * K);
        CHECK(!in_v(other));
        s.put(other);
        const size_t before = g_bytes, allocs = g_allocs;
        for (int i = 0; i < 50; i += 2)                    // of half of them all, of one all but the last
            for (uint32_t j = 0; j < 33u - (i == 0); ++j) reinterpret_cast<uint32_t *>(v[i].p)[j] = 8 << 2 | 1;
        std::vector<HostBlock> w;
        for (int i = 0; i < 25; ++i) {
            w.push_back(s.get(64 * K));
            CHECK(w[i].p == other.p || (in_v(w[i]) && w[i].p != v[0].p));
        }
        CHECK(g_allocs == allocs);
        w.push_back(s.get(64 * K));
        CHECK(!in_v(w.back()) && g_allocs == allocs + 1);
        for (auto &x : w) s.put(x);
        for (int i = 0; i < 50; ++i)
            if (i % 2 || i == 0)
                for (uint32_t j = 0; j < 33; ++j) reinterpret_cast<uint32_t *>(v[i].p)[j] = 8 << 2;
        HostBlock last = s.get(64 * K);
        s.put_when(last, 0, 0, 0);                         // (nothing to wait for)
        CHECK(g_bytes - before + 51 * 64 * K <= Store::kKeepBytes + 64 * K);
    }
    {
        // the same from several threads, another one writing the words
        static Store s;
        std::mutex lock;
        std::vector<unsigned char *> todo;
        bool stop = false;
        std::thread gpu([&] {
            for (;;) {
                std::vector<unsigned char *> now;
                {
                    std::lock_guard<std::mutex> hold(lock);
                    if (stop && todo.empty()) return;
                    now.swap(todo);
                }
                for (unsigned char *p : now)
                    for (uint32_t j = 0; j < 5; ++j) __atomic_store_n(reinterpret_cast<uint32_t *>(p) + j, 9 << 2, __ATOMIC_RELAXED);
            }
        });
        std::vector<std::thread> threads;
        for (unsigned t = 0; t < 3; ++t)
            threads.emplace_back([&] {
                for (int i = 0; i < 3000; ++i) {
                    HostBlock b = s.get(64 * K);
                    CHECK(b.p && __atomic_load_n(reinterpret_cast<uint32_t *>(b.p), __ATOMIC_RELAXED) != 1);   // (1: in use)
                    for (uint32_t j = 0; j < 5; ++j) __atomic_store_n(reinterpret_cast<uint32_t *>(b.p) + j, 1, __ATOMIC_RELAXED);
                    {
                        std::lock_guard<std::mutex> hold(lock);
                        todo.push_back(b.p);
                    }
                    s.put_when(b, 5, 9 << 2, ~3u);
                }
            });
        for (auto &th : threads) th.join();
        {
            std::lock_guard<std::mutex> hold(lock);
            stop = true;
        }
        gpu.join();
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
