// Host-side view of the library's internals for the CPU tests: the launch plans (bla_api.hip) and
// the slot order of the folded kernels (bla_device.h).  Compiled for the host only.
#include <stdio.h>
#include <stdlib.h>

#include "bla_api.hip"
#include "bla_device.h"

// plan: reads lines "form B H L d M S bf16 chunk anchor", form f (forward), b (backward) or s (step),
// with T = (1 + h mod 2)(2M - 1); prints the table key, where the tables and the scratch lie, and the
// work split.
static int plans()
{
    char form;
    int B, H, L, d, M, S, bf16, chunk, anchor;
    while (scanf(" %c %d %d %d %d %d %d %d %d %d", &form, &B, &H, &L, &d, &M, &S, &bf16, &chunk, &anchor) == 10) {
        bla_params p;
        memset(&p, 0, sizeof(p));
        p.B = B, p.H = H, p.L = L, p.d_k = p.d_v = d, p.M = M, p.S = S, p.chunk = chunk;
        p.io_dtype = bf16 ? BLA_BF16 : BLA_F32, p.phase_anchor = anchor;
        const bool step = form == 's';
        if ((form == 'b' ? check_backward_shape(&p) : check_shape(&p, step)) != BLA_OK) {
            printf("unsupported\n");
            continue;
        }
        double* T = (double*)malloc(sizeof(double) * H);
        for (int h = 0; h < H; ++h) T[h] = (1 + h % 2) * (2.0 * M - 1.0);
        Plan pl;
        if (form == 'b') {
            BwdPlan bp;
            make_bwd_plan(&p, &bp);
            pl = bp.pl;
        } else {
            make_plan(&p, step, &pl);
        }
        printf("key %llu summ %zu total %zu nseg %d cps %d pair %d fragtab %d tables", (unsigned long long)table_key(pl, T, step),
               pl.off_summ, pl.total, pl.nseg, pl.cps, pl.pair, pl.fragtab);
        const size_t offs[] = {pl.off_E32, pl.off_EbarT, pl.off_ErevT, pl.off_Etab, pl.off_ABs, pl.off_ABm, pl.off_theta,
                               pl.off_rotblk, pl.off_trig, pl.off_rperiod, pl.off_period, pl.off_fABs, pl.off_fABm,
                               pl.off_fEtab, pl.off_fEbar, pl.off_fErev, pl.off_fTw};
        for (size_t x : offs) printf(" %zu", x);
        printf("\n");
        free(T);
    }
    return 0;
}

// records: reads lines "build dev at bytes key" (a call whose tables, of `bytes` at address `at`, are
// built; it writes nothing else), "keep dev at n key" (a call that writes n bytes and would keep its
// tables; prints whether they are there) and "write dev at n" (one without tables).
static int records()
{
    char op[8];
    int dev;
    unsigned long long at, n, key;
    while (scanf(" %7s %d %llu %llu", op, &dev, &at, &n) == 4) {
        if (!strcmp(op, "write")) {
            tables_claim(dev, (const char*)at, n, nullptr);
            continue;
        }
        if (scanf("%llu", &key) != 1) return 1;
        const uint64_t k = key;
        const bool found = tables_claim(dev, (const char*)at, n, &k);
        if (!strcmp(op, "keep"))
            printf("%d\n", found);
        else
            tables_record(dev, (const char*)at, n, k);
    }
    return 0;
}

// slots: for every padded count SP of the folded kernels and slot count S that pads to it, a line "SP S"
// and the slots of the SP folded entries.
static int slots()
{
    for (int SP = 64; SP <= 256; SP *= 2)
        for (int S = SP / 2 + 1; S <= SP; ++S) {
            printf("%d %d", SP, S);
            for (int i = 0; i < SP; ++i) printf(" %d", folded_slot(i, S, SP));
            printf("\n");
        }
    return 0;
}

// products: reads lines "m n k"; prints whether the library's own kernel forms that product.
static int products()
{
    long long m, n, k;
    while (scanf("%lld %lld %lld", &m, &n, &k) == 3) printf("%d\n", gemm_takes(m, n, k));
    return 0;
}

int main(int argc, char** argv)
{
    if (argc == 2 && !strcmp(argv[1], "products")) return products();
    if (argc == 2 && !strcmp(argv[1], "slots")) return slots();
    if (argc == 2 && !strcmp(argv[1], "records")) return records();
    if (argc == 2 && !strcmp(argv[1], "plan")) return plans();
    return 2;
}
