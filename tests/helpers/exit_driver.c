/* A program that closes its simulation when the process ends, in a handler
 * registered before its first call into the library: the handler runs after
 * everything that was registered later. */
#include <stdio.h>
#include <stdlib.h>

#include "rdos.h"

static rdos_sim *sim;

static void at_end(void)
{
    rdos_destroy(sim);
    printf("closed\n");
    fflush(stdout);
}

int main(void)
{
    static const double xyz[15] = {0, 0, 0, 1e-6, 0, 0, 0, 1e-6, 0, 0, 0, 1e-6, 1e-6, 1e-6, 1e-6};
    static const int32_t tets[8] = {0, 1, 2, 3, 1, 2, 3, 4};
    int32_t species, counts[2] = {7, 2}, back[2];
    double tau;
    atexit(at_end);
    if (rdos_create(&sim, 0, 1, 1) != RDOS_OK || rdos_set_mesh(sim, 5, xyz, 2, tets) != RDOS_OK ||
        rdos_add_species(sim, 1e-12, &species) != RDOS_OK)
        return 1;
    if (rdos_finalize(sim, 1.0, &tau) != RDOS_OK || rdos_set_counts(sim, 0, 0, counts) != RDOS_OK) {
        fprintf(stderr, "%s\n", rdos_last_error(sim));
        return 2;
    }
    for (int i = 0; i < 8; ++i)  /* often enough for a pinned buffer to be made */
        if (rdos_get_counts(sim, 0, 0, back) != RDOS_OK || back[0] != 7 || back[1] != 2) return 3;
    return 0;
}
