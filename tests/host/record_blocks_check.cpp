// Host-only checks of the places of the server's group records
// (server_admission.hpp).  Exit status 1 on any failure.
#include <cstdio>

#include "server_admission.hpp"

int main()
{
    // the records of a mesh of every size take a multiple of 8 doubles; odd lengths
    // must not matter either
    int failures = 0;
    for (size_t first = 1; first < 3000; first += 7) {
        nebem::RecordBlocks b;
        size_t end = 0;
        for (size_t n = first, k = 0; k < 5; ++k, n = n * 3 % 1777 + 1) {
            const size_t at = b.add(n);
            if (at % 32 || at < end || b.len < at + n || b.len % 32) ++failures;
            end = at + n;
        }
        if (b.len > end + 31) ++failures;
    }
    std::printf("%s\n", failures ? "FAIL" : "checks passed");
    return failures != 0;
}
