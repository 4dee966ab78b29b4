// Prints numbers of next_nonce() for tests/test_nonce.py, from the kernel's
// entropy or (-DNO_ENTROPY) without it.
#include <cstddef>
#include <cstdio>
#include <sys/random.h>
#include <unistd.h>

#ifdef NO_ENTROPY
static int no_entropy(void*, size_t) noexcept { return -1; }
#define getentropy no_entropy
#endif

#include "../../paper_2607_04206_amd/csrc/nonce.h"

static_assert(noexcept(sangam::next_nonce()), "called from C entry points");

int main() {
    for (int i = 0; i < 1000; ++i) std::printf("%llx\n", (unsigned long long)sangam::next_nonce());
    return 0;
}
