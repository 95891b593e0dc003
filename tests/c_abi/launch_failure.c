/*
 * What a step that takes two launches leaves when one of them fails.  Needs no
 * GPU (hip_stub.h).  Test infrastructure only.
 */
#include "hip_stub.h"

static int fails;
static void check(int ok, const char *what)
{
    if (!ok) {
        printf("FAILED: %s\n", what);
        ++fails;
    }
}
int main(void)
{
    agft_config c;
    memset(&c, 0, sizeof(c));
    c.B = 8192;   /* the smallest batch that takes the separate update */
    c.K = 128;
    c.d = 16;
    c.lambda = 1.0f;
    c.alpha0 = 0.5f;
    c.prune_period = 50;
    c.prune_sticky = 1;
    /* device addresses: never read or written here */
    void *state = (void *)0x100000000ull;
    float *ctx = (float *)0x10000, *reward = (float *)0x20000, *scores = (float *)0x30000;
    int32_t *action = (int32_t *)0x40000;
    agft_handle *h = NULL;
    agft_state_view v;
#define T() (agft_get_state(h, &v), (int)v.t)
#define PENDING() (agft_get_state(h, &v), v.pending)
    start(0);
    check(agft_create(&c, state, agft_state_bytes(&c), NULL, &h) == AGFT_OK && n_ran == 1, "set-up");
    start(0);
    check(agft_step(h, ctx, NULL, action, NULL) == AGFT_OK && n_ran == 1, "first step: one launch");
    const void *one = ran[0];
    start(0);
    check(agft_step(h, ctx, reward, action, NULL) == AGFT_OK && n_ran == 2, "second step: update and score");
    const void *update = ran[0], *score = ran[1];
    check(update != score && score != one, "kernels of their own");

    start(2);
    check(agft_step(h, ctx, reward, action, NULL) == AGFT_E_HIP, "score launch fails");
    check(n_ran == 1 && ran[0] == update && T() == 2 && PENDING() == 1, "the decision is not made");
    start(0);
    check(agft_step(h, ctx, reward, action, NULL) == AGFT_OK && n_ran == 1 && ran[0] == score && T() == 3,
          "called again: the reward is not folded in again");
    start(0);
    check(agft_step(h, ctx, reward, action, NULL) == AGFT_OK && n_ran == 2 && ran[0] == update, "the next step as ever");

    start(1);
    check(agft_step(h, ctx, reward, action, NULL) == AGFT_E_HIP && n_ran == 0 && T() == 4, "update launch fails");
    start(0);
    check(agft_step(h, ctx, reward, action, NULL) == AGFT_OK && n_ran == 2 && ran[0] == update, "called again: whole step");

    start(2);
    check(agft_step(h, ctx, reward, action, NULL) == AGFT_E_HIP, "score launch fails again");
    start(0);
    check(agft_step(h, ctx, reward, action, scores) == AGFT_OK && n_ran == 1 && ran[0] == score, "called again for the scores");

    start(0);
    check(agft_step(h, NULL, reward, NULL, NULL) == AGFT_OK && n_ran == 1 && ran[0] == one && PENDING() == 0, "flush");
    start(0);
    check(agft_step(h, ctx, NULL, action, NULL) == AGFT_OK && n_ran == 1 && ran[0] == one, "a step with nothing pending");
    start(2);
    check(agft_step(h, ctx, reward, action, NULL) == AGFT_E_HIP, "score launch fails before a flush");
    start(0);
    check(agft_step(h, NULL, reward, NULL, NULL) == AGFT_OK && n_ran == 1 && ran[0] == score && PENDING() == 0,
          "flush: the reward is not folded in again");
    start(0);
    check(agft_step(h, ctx, NULL, action, NULL) == AGFT_OK && n_ran == 1 && ran[0] == one, "a step after that flush");

    /* the simulator's step on such a handle: the score kernel, then the environment's */
    agft_env_config e;
    memset(&e, 0, sizeof(e));
    e.B = c.B, e.K = c.K, e.d = c.d, e.T = 1000;
    e.P0 = e.c = e.l0 = e.a = e.b = 1.0f;
    e.lat_min = e.f_lo = 0.1f, e.f_hi = 1.0f, e.f_init = 0.5f, e.tpot_div = 1.0f;
    e.svc_lo = e.svc_hi = e.svc_init = 4;
    e.q_cap = e.run_cap = 100;
    for (int i = 0; i < 7; ++i) e.sd[i] = 1.0f;
    const size_t ne = agft_env_state_bytes(&e);
    check(ne > 0, "environment configuration");
    start(0);
    check(agft_sim_step(h, &e, (void *)0x200000000ull, ne, (int32_t *)0x50000, (float *)0x60000, ctx, reward, action, NULL) ==
              AGFT_OK && n_ran == 3 && ran[0] == update && ran[1] == score, "simulator step: three launches");
    start(2);
    check(agft_step(h, ctx, reward, action, NULL) == AGFT_E_HIP, "score launch fails before a simulator step");
    start(0);
    check(agft_sim_step(h, &e, (void *)0x200000000ull, ne, (int32_t *)0x50000, (float *)0x60000, ctx, reward, action, NULL) ==
              AGFT_OK && n_ran == 2 && ran[0] == score, "simulator step: the reward is not folded in again");
    check(agft_destroy(h) == AGFT_OK, "destroy");

    /* a buffer saved between the two launches: the update marks its header (pending = 2) */
    c.flags = AGFT_ADOPT_STATE;
    for (int32_t pending = 0; pending <= 3; ++pending) {
        memcpy(header + 28, &pending, 4);
        start(0);
        const int rc = agft_create(&c, state, agft_state_bytes(&c), NULL, &h);
        check(rc == (pending == 3 ? AGFT_E_STATE : AGFT_OK), "adopt");
        if (rc != AGFT_OK) continue;
        check(PENDING() == (pending != 0), "adopted: pending");
        check(agft_step(h, ctx, reward, action, NULL) == AGFT_OK && n_ran == (pending == 1 ? 2 : 1) &&
                  ran[0] == (pending == 0 ? one : pending == 1 ? update : score), "adopted: first step");
        check(agft_destroy(h) == AGFT_OK, "destroy");
    }
    printf("launch failure: %d failures\n", fails);
    return fails != 0;
}
