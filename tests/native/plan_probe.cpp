// Plans of calls, on the CPU: handles are filled in by hand, nothing is
// enqueued and no device is touched.  Reads one call per line from stdin and
// writes one line each (see tests/test_plans.py):
//   batch R C pitch aligned B modulus m variant  ->  status name splits kts need workspace
// m > 0: the call gathers m rows; variant: pinned for B's bucket (0: none).
//   noalloc R C pitch aligned B  ->  status name splits kts need, of the allocation-free call
//   fit R C pitch aligned B modulus scratch  ->  name splits kts need, cut to a scratch
//   kept R C pitch aligned B modulus other  ->  names of the plans of B, of B mod
//                           p, of `other` and of the first two again, on one handle
//   answer R C pitch aligned 0  ->  name row_blocks splits threads, of the single query
//   few R C pitch aligned B  ->  rows_per_block splits, of the dot4 stream
#include <cstdio>
#include <cstring>
#include <memory>

#include "qpir_internal.h"

static std::unique_ptr<pir_db> handle(uint64_t R, uint64_t C, uint64_t pitch, int aligned) {
    std::unique_ptr<pir_db> db(new pir_db());
    db->magic = kDbMagic;
    db->D = reinterpret_cast<uint8_t*>(uintptr_t{4096});
    db->rows = R;
    db->cols = C;
    db->pitch = pitch;
    db->aligned = aligned != 0;
    gemv_open(db.get());
    return db;
}

int main() {
    char op[16];
    unsigned long long R, C, pitch;
    unsigned B, mod, m, v;
    int aligned;
    while (scanf("%15s %llu %llu %llu %d %u", op, &R, &C, &pitch, &aligned, &B) == 6) {
        const auto db = handle(R, C, pitch, aligned);
        if (strcmp(op, "batch") == 0) {
            if (scanf("%u %u %u", &mod, &m, &v) != 3) return 2;
            (m ? db->variant_rows : db->variant)[batch_bucket(B)] = (uint8_t)v;
            BatchPlan p{};
            const auto* rows = reinterpret_cast<const uint32_t*>(m ? uintptr_t{4096} : 0);
            const pir_status st = mfma_plan_batch(db.get(), B, rows, m, mod, false, &p);
            printf("%d %s %u %u %zu %zu\n", (int)st, mfma_variant_name(p.variant), p.splits, p.kts,
                   p.need, mfma_workspace_bytes(db.get(), B));
        } else if (strcmp(op, "noalloc") == 0) {
            BatchPlan p{};
            pir_status st = mfma_plan_batch(db.get(), B, nullptr, 0, 0, false, &p);
            if (st == PIR_OK) {
                mfma_plan_fit(db.get(), B, PIR_NOALLOC_SCRATCH_BYTES, &p);
                if (p.need > PIR_NOALLOC_SCRATCH_BYTES) st = PIR_ERR_SHAPE;
            }
            printf("%d %s %u %u %zu\n", (int)st, mfma_variant_name(p.variant), p.splits, p.kts, p.need);
        } else if (strcmp(op, "fit") == 0) {
            unsigned long long scratch;
            if (scanf("%u %llu", &mod, &scratch) != 2) return 2;
            BatchPlan p{};
            if (mfma_plan_batch(db.get(), B, nullptr, 0, mod, false, &p) != PIR_OK) return 3;
            mfma_plan_fit(db.get(), B, scratch, &p);
            printf("%s %u %u %zu\n", mfma_variant_name(p.variant), p.splits, p.kts, p.need);
        } else if (strcmp(op, "kept") == 0) {
            unsigned other;
            if (scanf("%u %u", &mod, &other) != 2) return 2;
            const unsigned Bs[] = {B, B, other, B, B}, ms[] = {0, mod, 0, 0, mod};
            for (int i = 0; i < 5; ++i) {
                BatchPlan p{};
                const pir_status st = mfma_plan_batch(db.get(), Bs[i], nullptr, 0, ms[i], false, &p);
                printf("%d:%s ", (int)st, mfma_variant_name(p.variant));
            }
            printf("\n");
        } else if (strcmp(op, "answer") == 0) {
            const GemvPlan p = gemv_plan(db.get());
            printf("%s %u %u %u\n", gemv_variant_name(p.variant), p.row_blocks, p.splits, p.threads);
        } else if (strcmp(op, "few") == 0) {
            const FewPlan p = few_batch_plan(db.get(), B);
            printf("%u %u\n", p.rows_per_block, p.splits);
        } else {
            return 2;
        }
    }
    return 0;
}
