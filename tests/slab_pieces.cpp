// Slab of pdhg_internal.hpp with an allocator that only records: allocations of
// the push model stay below two megabytes where each array does, are one
// otherwise, and hold every array whole and apart from the others.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <vector>

struct Block {
    uintptr_t base;
    size_t bytes;
};
static std::vector<Block> blocks;
static hipError_t record(void **p, size_t bytes)
{
    const uintptr_t base = blocks.empty() ? 1 << 20 : (blocks.back().base + blocks.back().bytes + 8191) / 4096 * 4096;
    blocks.push_back({base, bytes});
    *p = reinterpret_cast<void *>(base);
    return hipSuccess;
}
#define hipMalloc(p, bytes) record((void **)(p), bytes)
#include "pdhg_internal.hpp"

static int check(const char *name, const std::vector<size_t> &bytes, size_t want_blocks)
{
    blocks.clear();
    pdhg::Slab slab;
    std::vector<char *> p(bytes.size());
    std::vector<void *> bases;
    for (size_t k = 0; k < bytes.size(); k++) slab.add(&p[k], bytes[k]);
    if (slab.commit_small(&bases) != hipSuccess) return 1;
    bool ok = blocks.size() == want_blocks && bases.size() == want_blocks;
    for (size_t b = 0; ok && b < blocks.size(); b++)
        ok = reinterpret_cast<uintptr_t>(bases[b]) == blocks[b].base && (want_blocks == 1 || blocks[b].bytes < (2u << 20));
    uintptr_t end = 0;
    for (size_t k = 0; ok && k < p.size(); k++) { // in the order of the adds, inside one block each
        const uintptr_t a = reinterpret_cast<uintptr_t>(p[k]);
        bool inside = false;
        for (const Block &b : blocks) inside = inside || (a >= b.base && a + bytes[k] <= b.base + b.bytes);
        ok = inside && a >= end && a % 256 == 0;
        end = a + bytes[k];
    }
    if (!ok) printf("%s: %zu blocks, %zu wanted\n", name, blocks.size(), want_blocks);
    return ok ? 0 : 1;
}

int main()
{
    const size_t mb = 1 << 20;
    int bad = 0;
    bad += check("three below, together above", {mb + 1, mb + 1, mb + 1}, 3);
    bad += check("two share a block", {mb - 256, mb - 256, mb, 5}, 2);
    bad += check("all in one", {0, 1, 255, 256, 257, mb / 2}, 1);
    bad += check("the last below the line", {2 * mb - 256}, 1);
    bad += check("one at the line", {mb, 2 * mb, mb}, 1);
    bad += check("a large one among small", {3, 64 * mb, mb, mb, mb, 7}, 1);
    return bad;
}
