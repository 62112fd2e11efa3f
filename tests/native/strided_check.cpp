// strided_check.cpp -- the compact program of regular layouts
// (locate_strided) against the general one (locate_any), position by
// position, on the host: random nests of loops over one run, negative and
// wide strides, spans of one byte, resized and wide extents, sizes up to and
// past the 32-bit limits, one element and counts.
#include <cinttypes>
#include <cstdio>
#include <random>

#include "core.h"
#include "mdt.h"

using namespace mdt;

static std::mt19937_64 g_rng(20240219);
static int64_t pick(int64_t lo, int64_t hi) { return lo + (int64_t)(g_rng() % (uint64_t)(hi - lo + 1)); }

static mdt_type keep(mdt_type t, int rc, mdt_type old)
{
    if (rc != MDT_SUCCESS) return old;
    if (old) mdt_type_free(&old);  // predefined handles refuse, which is fine
    return t;
}

static mdt_type random_type(bool big)
{
    mdt_type t = mdt_basic((int)pick(0, MDT_NUM_BASIC - 1)), n = nullptr;
    const int depth = (int)pick(1, 6);
    for (int d = 0; d < depth; d++) {
        const int64_t cnt = big && d == 0 ? pick(1, 1 << 22) : pick(1, big ? 60 : 9);
        mdt_aint lb, ext;
        mdt_type_get_extent(t, &lb, &ext);
        switch (pick(0, 5)) {
        case 0: t = keep(n, mdt_type_contiguous(cnt, t, &n), t); break;
        case 1: t = keep(n, mdt_type_vector(cnt, pick(1, 5), pick(-8, 12), t, &n), t); break;
        case 2:
            t = keep(n, mdt_type_create_hvector(cnt, pick(1, 3),
                                                pick(0, 9) ? pick(-300, 900) : pick(-4000000000ll, 4000000000ll), t, &n), t);
            break;
        case 3: {
            mdt_count s[3], u[3], b[3];
            for (int i = 0; i < 3; i++) {
                s[i] = pick(1, big ? 40 : 7);
                u[i] = pick(1, s[i]);
                b[i] = pick(0, s[i] - u[i]);
            }
            t = keep(n, mdt_type_create_subarray(3, s, u, b, (int)pick(0, 1), t, &n), t);
            break;
        }
        case 4: {
            const mdt_count gs[3] = {pick(1, 40), pick(1, 40), pick(1, 40)};
            const int di[3] = {MDT_DISTRIBUTE_CYCLIC, MDT_DISTRIBUTE_CYCLIC, MDT_DISTRIBUTE_CYCLIC};
            const int da[3] = {(int)pick(1, 5), (int)pick(1, 5), (int)pick(1, 5)}, ps[3] = {2, 2, 2};
            // ranks whose share is ragged in every dimension or in none
            t = keep(n, mdt_type_create_darray(8, pick(0, 1) ? 7 : 0, 3, gs, di, da, ps, MDT_ORDER_C, t, &n), t);
            break;
        }
        default: t = keep(n, mdt_type_create_resized(t, 0, pick(0, 7) ? ext + pick(0, 64) : ext + (3ll << 30), &n), t);
        }
        mdt_count size;
        mdt_type_size(t, &size);
        if (size > ((mdt_count)1 << 32)) break;
    }
    return t;
}

int main()
{
    int64_t types = 0, on = 0, checked = 0, multi = 0, bad = 0;
    for (int it = 0; it < 6000; it++) {
        mdt_type h = random_type(it % 3 == 0);
        mdt_count size;
        mdt_type_size(h, &size);
        if (size > 0 && size < ((mdt_count)1 << 33) && mdt_type_commit(&h) == MDT_SUCCESS) {
            types++;
            const DevLayout &L = reinterpret_cast<TypeNode *>(h)->comp->host;
            const DevStrided &S = L.st;
            if (S.on) {
                on++;
                multi += L.kind == KIND_MULTI;
                for (int k = 0; k < 200; k++) {
                    const bool elem1 = S.elem1_only || pick(0, 1);
                    const uint64_t p = elem1 ? (uint64_t)pick(0, size - 1) : (uint64_t)pick(0, 5 * size - 1);
                    uint32_t rel = (uint32_t)pick(0, 65535);
                    if (elem1 && p + rel >= (uint64_t)size) rel = (uint32_t)(size - 1 - (int64_t)p);
                    const Loc want = locate_any(L, p + rel);
                    // as a tile does: the first byte in 64 bits, the rest in 32
                    const uint64_t e = elem1 ? 0 : magic_div(p, S.dsize);
                    const Loc32 got = locate_strided(S, (uint32_t)(p - e * S.size) + rel, S.base + (int64_t)e * S.extent, elem1);
                    checked++;
                    if (got.addr != want.addr || got.rem != want.rem) {
                        if (bad++ < 5)
                            std::fprintf(stderr, "p %" PRIu64 " + %u: (%" PRId64 ", %d), general (%" PRId64 ", %" PRId64 ")\n", p,
                                         rel, got.addr, got.rem, want.addr, want.rem);
                    }
                }
            }
        }
        mdt_type_free(&h);
    }
    std::printf("%lld types, %lld compact (%lld with outer loops), %lld positions, bad %lld\n", (long long)types,
                (long long)on, (long long)multi, (long long)checked, (long long)bad);
    return bad || on < 500 || multi < 10;
}
