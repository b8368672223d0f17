// Host-only checks of the places of the server's group records
// (server_admission.hpp).  Exit status 1 on any failure.
#include <cstdio>

#include "server_admission.hpp"

int main()
{
    // geometries' blocks follow each other without overlap, whatever their lengths,
    // and so do the two streams' sets of len doubles
    int failures = 0;
    for (size_t first = 1; first < 3000; first += 7) {
        nebem::RecordBlocks b;
        size_t end = 0;
        for (size_t n = first, k = 0; k < 5; ++k, n = n * 3 % 1777 + 1) {
            const size_t at = b.add(n);
            if (at < end || b.len < at + n) ++failures;
            end = at + n;
        }
        if (b.len > end + 4) ++failures;
    }
    std::printf("%s\n", failures ? "FAIL" : "checks passed");
    return failures != 0;
}
