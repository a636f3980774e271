// Prints scatter_grid(round, entries, units, bytes) for every line of four numbers on its input.
#include <cstdio>

#include "launch_rules.hpp"

int main() {
    long long round, entries, units, bytes;
    while (std::scanf("%lld %lld %lld %lld", &round, &entries, &units, &bytes) == 4)
        std::printf("%lld\n", (long long)ptsd::scatter_grid(round, entries, units, bytes));
    return 0;
}
