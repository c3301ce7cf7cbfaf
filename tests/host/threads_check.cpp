// Prints, for each count of slot-BP workgroups on a compute unit that the library launches, their threads.
#include <cstdio>

#include "qlsd_internal.h"

int main() {
    for (int wg : {1, 2, 3, 4, 5, 6, 8}) printf("%d %d ", wg, qlsd::bp_threads_for(wg));
    return 0;
}
