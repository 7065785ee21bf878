// ensure_pinned (csrc/pinned.h) with calls that fail on demand: what a failed first use leaves behind.
#include <stdio.h>
#include <stdlib.h>

#include "../../paper_2604_03446_amd/csrc/pinned.h"

static int fail_alloc, fail_address, held;

struct FakeApi {
    int success = 0;
    int alloc(unsigned char **p, size_t bytes) const
    {
        if (fail_alloc) return 2;
        *p = (unsigned char *)malloc(bytes);
        ++held;
        return 0;
    }
    int address(unsigned char **map, unsigned char *host) const
    {
        if (fail_address) return 7;
        *map = host;
        return 0;
    }
    int release(unsigned char *host) const { free(host); --held; return 0; }
};

#define CHECK(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

int main()
{
    mmee::Pinned m;
    fail_alloc = 1;
    CHECK(mmee::ensure_pinned(FakeApi{}, m, 64) == 2 && !m.host && !m.map && held == 0);
    fail_alloc = 0; fail_address = 1;
    CHECK(mmee::ensure_pinned(FakeApi{}, m, 64) == 7 && !m.host && !m.map && held == 0);
    CHECK(mmee::ensure_pinned(FakeApi{}, m, 64) == 7 && !m.host && !m.map && held == 0);   // not remembered as done
    fail_address = 0;
    CHECK(mmee::ensure_pinned(FakeApi{}, m, 64) == 0 && m.host && m.map && held == 1);
    unsigned char *kept = m.host;
    fail_alloc = fail_address = 1;
    CHECK(mmee::ensure_pinned(FakeApi{}, m, 64) == 0 && m.host == kept && held == 1);      // there already
    free(m.host);
    printf("ok\n");
    return 0;
}
