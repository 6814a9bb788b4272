// Prints which kernel an automatic call takes, one line per input line:
//   kind (0 HEAL-Base, 1 HEAL-Full, 2 INT16 scores, 3 pre-split, 4 bf16x3 with B
//   stored K x N, 5 with B stored N x K), M, N, K, batch, extra elements per row
//   of A, of B and of C, and bytes by which A, B and C miss 16-byte alignment.
// Operands are dense but for the extra elements; nothing is dereferenced.
#include <cstdio>

#include "heal.h"
#include "heal_internal.h"

int main()
{
    long kind, M, N, K, batch, pa, pb, pc, oa, ob, oc;
    while (scanf("%ld %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld", &kind, &M, &N, &K, &batch, &pa, &pb, &pc, &oa,
                 &ob, &oc) == 11) {
        const int64_t lda = K + pa, ldb = (kind == 4 ? N : K) + pb, ldc = N + pc;
        const int64_t sa = M * lda, sb = (kind == 4 ? K : N) * ldb, sc = M * ldc;
        const int unit = kind == 2 ? 8 : 4;
        const char *base = reinterpret_cast<const char *>(0x100000);
        auto whole = [&](int64_t ld, int64_t stride, int u, long off) {
            return off == 0 && ld % u == 0 && (batch == 1 || stride % u == 0);
        };
        heal::Route r;
        if (kind >= 4) {
            heal::GemmArgs a = {};
            a.M = M; a.N = N; a.K = K; a.batch = batch;
            a.A = reinterpret_cast<const float *>(base + oa); a.lda = lda; a.strideA = sa;
            a.B = reinterpret_cast<const float *>(base + ob); a.ldb = ldb; a.strideB = sb;
            a.C = reinterpret_cast<float *>(const_cast<char *>(base + oc)); a.ldc = ldc; a.strideC = sc;
            a.alpha = 1.0f;
            a.vecA = whole(lda, sa, 4, oa); a.vecB = whole(ldb, sb, 4, ob); a.vecC = whole(ldc, sc, 4, oc);
            r = heal::choose_gemm(a, kind == 5);
        } else {
            heal::OpArgs a = {};
            a.M = M; a.N = N; a.K = K; a.batch = batch;
            a.A = base + oa; a.lda = lda; a.strideA = sa;
            a.B = base + ob; a.ldb = ldb; a.strideB = sb;
            a.C = reinterpret_cast<float *>(const_cast<char *>(base + oc)); a.ldc = ldc; a.strideC = sc;
            a.vecA = whole(lda, sa, unit, oa); a.vecB = whole(ldb, sb, unit, ob); a.vecC = whole(ldc, sc, 4, oc);
            r = heal::choose_op((int)kind, a);
        }
        if (r.kernel == heal::ROUTE_PANEL) puts("panel");
        else if (r.kernel == heal::ROUTE_DIRECT) printf("direct %d\n", heal::direct_tile(r.plan));
        else puts(r.kernel == HEAL_INSTANCE_LARGE ? "large" : r.kernel == HEAL_INSTANCE_MEDIUM ? "medium" : "skinny");
    }
}
