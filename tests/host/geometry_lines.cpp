// Reads problems from standard input and prints the launch geometry that the library derives for them, one line per layer:
//   batch K v m g fp32 count N1 .. Ncount B0 [the eight fields of a plan, if B0 is 0]
// The plan is the default one of the summed height at batch B0, or the given one.  For each problem: a line "group STATUS", and per
// layer a line as a member of the group, when that is 0 (groups end at 32 rows), and one alone.
#include <cstdio>

#include "cg_common.h"

using namespace cg;

static void print(const char* what, const Geometry& g)
{
    std::printf("%s N=%d rows=%d staged=%d prompt=%d half=%d bg=%d nblk=%d nks=%d kpw=%d waves=%d build=%d words=%d pairs=%zu\n", what, g.N, g.RB, (int)g.staged,
                (int)g.prompt, (int)g.half, g.BG, g.NBLK, g.NKS, g.KPW, g.NW, g.NB, g.RPL, pair_words(g));
}

int main()
{
    codegemm_desc d = {};
    int fp32, count, n[kMaxGroup], plan_batch;
    while (std::scanf("%d %d %d %d %d %d %d", &d.batch, &d.in_features, &d.vec_len, &d.num_codebooks, &d.group_size, &fp32, &count) == 7) {
        d.code_bits = 8;
        d.flags = fp32 ? CODEGEMM_FLAG_Y_FP32 : 0;
        d.out_features = 0;
        if (count < 1 || count > kMaxGroup) return 1;
        for (int i = 0; i < count; ++i) {
            if (std::scanf("%d", &n[i]) != 1) return 1;
            d.out_features += n[i];
        }
        codegemm_plan p = {};
        if (std::scanf("%d", &plan_batch) != 1) return 1;
        if (plan_batch) {
            codegemm_desc other = d;
            other.batch = plan_batch;
            if (codegemm_default_plan(&other, &p)) return 2;
        } else {
            if (std::scanf("%d %d %d %d %d %d %d %d", &p.waves, &p.row_words, &p.k_splits, &p.batch_group, &p.psum_dtype, &p.build_waves, &p.centroid_rows,
                           &p.centroid_splits) != 8) return 1;
        }
        Geometry members[kMaxGroup], whole, alone;
        const int st = group_geometry(&d, &p, n, count, members, &whole);
        std::printf("group %d\n", st);
        for (int i = 0; i < count; ++i) {
            codegemm_desc one = d;
            one.out_features = n[i];
            if (st == 0) print("member", members[i]);
            if (make_geometry(&one, &p, &alone) == 0) print("alone", alone);
            else if (st == 0) return 3;
        }
    }
    return 0;
}
