/*
 * The launches of a step: for every line "CFG T DUMP" of the input (CFG the
 * bytes of an agft_config in hexadecimal), the launches of the decision after T
 * others, with (DUMP 1) or without the score dump, each as "threads per
 * workgroup x workgroups".  Needs no GPU (hip_stub.h).  Test infrastructure only.
 */
#include "hip_stub.h"

int main(void)
{
    static char hex[2 * sizeof(agft_config) + 2];
    int t, dump;
    /* device addresses: never read or written here */
    void *state = (void *)0x10000000000ull;
    float *ctx = (float *)0x10000, *reward = (float *)0x20000, *scores = (float *)0x30000;
    while (scanf("%233s %d %d", hex, &t, &dump) == 3) {
        agft_config c;
        unsigned char *bytes = (unsigned char *)&c;
        for (size_t i = 0; i < sizeof(c); ++i) {
            unsigned v;
            if (sscanf(hex + 2 * i, "%2x", &v) != 1) return 2;
            bytes[i] = (unsigned char)v;
        }
        agft_handle *h;
        if (agft_create(&c, state, agft_state_bytes(&c), NULL, &h) != AGFT_OK) return 3;
        for (int i = 0; i <= t; ++i) {
            start(0);
            if (agft_step(h, ctx, reward, NULL, i == t && dump ? scores : NULL) != AGFT_OK) return 4;
        }
        for (int i = 0; i < n_ran; ++i) printf("%s%ux%u", i ? " " : "", ran_block[i], ran_grid[i]);
        printf("\n");
        agft_destroy(h);
    }
    return 0;
}
