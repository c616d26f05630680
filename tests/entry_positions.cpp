// The row sums of pdhg_device.hpp and pdhg_kernels.hpp built for the host and
// run on rows whose entries are the last ones a model may hold (positions up to
// 2^31 - 2).  Only the pages of those entries are mapped; a position that wraps
// lands in reserved pages and ends the process.  Values are small integers, so
// every order of a sum gives the same number.  Lane groups run lane by lane, a
// ballot being the lane's own vote (rounds only differ in what they prefetch);
// a tile runs with one thread per lane and one lane per row.
#include <hip/hip_runtime.h>

#include <pthread.h>
#include <sys/mman.h>

#include <climits>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>

namespace host {
struct Index {
    unsigned x;
};
thread_local Index tid;
thread_local int lanes = 1; // threads that run the function together
pthread_barrier_t bar;
void sync()
{
    if (lanes > 1) pthread_barrier_wait(&bar);
}
} // namespace host

#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
#define threadIdx host::tid
#define __syncthreads() host::sync()
#define __builtin_amdgcn_ballot_w64(p) (p)
#include "pdhg_kernels.hpp"

constexpr int64_t kEnd = ((int64_t)1 << 31) - 1, kMapped = 65536;

template <typename T>
T *last_entries() // position 0 of an array of 2^31 with its last kMapped entries mapped, as much reserved before it
{
    const size_t size = sizeof(T) << 31, tail = sizeof(T) * kMapped;
    char *p = (char *)mmap(nullptr, 2 * size + (1 << 20), PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == (char *)MAP_FAILED || mprotect(p + 2 * size - tail, tail, PROT_READ | PROT_WRITE) != 0) exit(2);
    return (T *)(p + size);
}

int *idx;
double *val, x[1024];
int failures = 0;

double exact(int64_t beg, int64_t end)
{
    double s = 0.0;
    for (int64_t e = beg; e < end; e++) s += val[e] * x[idx[e]];
    return s;
}

void expect(const char *what, int64_t len, double got, double want)
{
    if (got == want) return;
    printf("%s, %lld entries: %.17g, expected %.17g\n", what, (long long)len, got, want);
    failures++;
}

template <int L>
void lane_groups()
{
    for (int64_t len : {0, 1, L, 4 * L - 1, 4 * L, 4 * L + 1, 8 * L, 8 * L + 1, 17 * L + 3, 41 * L}) {
        const int64_t beg = kEnd - len;
        double s = 0.0;
        for (int lane = 0; lane < L; lane++) s += pdhg::lane_dot<L, double>((int)beg, (int)kEnd, lane, idx, val, x);
        expect("lane group", len, s, exact(beg, kEnd));
    }
}

// rows of `longest` entries and less that end with the last entry
std::vector<int> rows_of(int rows, int longest)
{
    std::mt19937 rng(rows + longest);
    std::vector<int> ptr(rows + 1, (int)kEnd);
    for (int r = rows; r > 0; r--) ptr[r - 1] = ptr[r] - (int)(rng() % (longest + 1));
    return ptr;
}

template <typename F>
void together(int n, F f)
{
    pthread_barrier_init(&host::bar, nullptr, n);
    std::vector<std::thread> t;
    for (int k = 0; k < n; k++)
        t.emplace_back([=] {
            host::tid.x = k;
            host::lanes = n;
            f(k);
        });
    for (auto &q : t) q.join();
    pthread_barrier_destroy(&host::bar);
}

void tiles(int longest)
{
    const std::vector<int> p = rows_of(256, longest);
    std::vector<int> s_ptr(257);
    std::vector<double> s_prod(pdhg::kTileU * 256), sum(256);
    const int *ptr = p.data();
    int *sp = s_ptr.data();
    double *pr = s_prod.data(), *su = sum.data();
    together(256, [=](int) {
        pdhg::TileRange r;
        r.beg = ptr[0];
        r.end = ptr[256];
        pdhg::tile_row_sums<double, double, 256, 256>(r, 0, 256, ptr, idx, val, x, sp, pr, su);
    });
    for (int r = 0; r < 256; r++) expect("tile row", p[r + 1] - p[r], sum[r], exact(p[r], p[r + 1]));
}

// one wave per few rows only while the positions that run ahead of the last entry stay below 2^31
void rule()
{
    pdhg_solver s;
    s.m = s.n = 1000;
    s.longest_row = s.longest_col = 4;
    for (int ahead : {0, pdhg::kWaveAhead - 1, pdhg::kWaveAhead, 1 << 20}) {
        s.nnz = (int)(kEnd - ahead);
        for (int kern : {-32, -64, -256})
            expect("waves for a model", s.nnz, pdhg::uses_waves(&s, kern, true), ahead >= pdhg::kWaveAhead);
    }
}

int main()
{
    idx = last_entries<int>();
    val = last_entries<double>();
    std::mt19937 rng(1);
    for (int64_t e = kEnd - kMapped + 1; e < kEnd; e++) {
        idx[e] = (int)(rng() % 1024);
        val[e] = (double)(int)(rng() % 17) - 8.0;
    }
    for (double &v : x) v = (double)(int)(rng() % 17) - 8.0;
    setvbuf(stdout, nullptr, _IONBF, 0);
    printf("lane groups\n");
    lane_groups<1>();
    lane_groups<8>();
    lane_groups<64>();
    for (int longest : {3, 8, 16, 40}) {
        printf("tiles of rows up to %d\n", longest);
        tiles(longest);
    }
    rule();
    printf("%d failures\n", failures);
    return failures ? 1 : 0;
}
