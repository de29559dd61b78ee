// Prints what the library's host-side plan rules decide, for queries read from
// stdin, one line each: a context of 256 CUs that launches nothing.
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "nbreg.h"
#include "nb_internal.h"
#include "nb_runtime.h"

int main()
{
    nb_ctx ctx;
    ctx.cu_count = 256;
    char what[32];
    while (std::scanf("%31s", what) == 1) {
        if (!std::strcmp(what, "plan")) {   // n n_i mixed
            long long n, n_i, mixed;
            if (std::scanf("%lld %lld %lld", &n, &n_i, &mixed) != 3) return 1;
            nb::Plan p = nbrt::auto_plan(&ctx, n, (int32_t)n_i, mixed != 0);
            int64_t len = 0;
            nbrt::finish_plan(p, n, (int32_t)n_i, &len);
            std::printf("%d %d %d %lld\n", p.mapping, p.rows_per_lane, p.splits, (long long)len);
        } else if (!std::strcmp(what, "redo")) {   // n n_i rows_per_item
            long long n, n_i, per;
            if (std::scanf("%lld %lld %lld", &n, &n_i, &per) != 3) return 1;
            nb::ForceArgs a{};
            a.n = n;
            a.n_i = (int32_t)n_i;
            int32_t words[64] = {};
            nb::bind_redo_scratch(a, nullptr, words, nb::redo_groups_for(ctx.cu_count), n);
            std::printf("%d %d\n", nb::redo_grid(a, (int)per), nb::redo_groups_for(ctx.cu_count));
        } else if (!std::strcmp(what, "fit")) {   // n n_i mixed budget fixed
            long long n, n_i, mixed, budget, fixed;
            if (std::scanf("%lld %lld %lld %lld %lld", &n, &n_i, &mixed, &budget, &fixed) != 5)
                return 1;
            const nb::Plan p = nbrt::auto_plan(&ctx, n, (int32_t)n_i, mixed != 0);
            const int least = fixed ? 1 : nbrt::least_splits(&ctx, n, (int32_t)n_i, p);
            const nbrt::ForceScratch f = nbrt::fit_scratch(&ctx, n, (int32_t)n_i, p,
                                                           mixed && !p.f64, least, (size_t)budget);
            std::printf("%d %lld %lld %d %d\n", f.p.splits, (long long)f.split_len,
                        (long long)f.total(), f.pack > 0, f.least);
        } else if (!std::strcmp(what, "adjoint")) {   // n n_i budget (0: any)
            long long n, n_i, budget;
            if (std::scanf("%lld %lld %lld", &n, &n_i, &budget) != 3) return 1;
            const nb::AdjointShape sh = nb::adjoint_shape(n, (int32_t)n_i, ctx.cu_count,
                                                          budget ? (size_t)budget : SIZE_MAX);
            std::printf("%d %d %lld %lld %d %lld\n", sh.row_block, sh.tile, (long long)sh.body_len,
                        (long long)sh.panel_blocks, sh.index_in_gm,
                        (long long)nb::adjoint_scratch_bytes(n, (int32_t)n_i, sh));
        } else if (!std::strcmp(what, "tune")) {   // n n_i mixed: candidates, first mapping
            long long n, n_i, mixed;
            if (std::scanf("%lld %lld %lld", &n, &n_i, &mixed) != 3) return 1;
            const auto c = nbrt::tune_candidates(&ctx, n, (int32_t)n_i, mixed != 0);
            int automatic = 0;
            for (const nb::Plan &p : c) automatic += p.mapping == 0;
            std::printf("%d %d %d\n", (int)c.size(), c[0].mapping, automatic);
        } else {
            return 1;
        }
    }
    return 0;
}
