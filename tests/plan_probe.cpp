// Prints which kernels a plan sends its passes to, and what the plan's self-check says of it and of mistakes planted in it, for
// tests/test_plan_routes.py (host code only; built there with the library's plan.cpp).  Arguments: kind (step, rows, columns), rank,
// bits, block, dtype, then rows and columns of every matrix (and, for the sketches, its buckets).
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "plan.h"

int main(int argc, char **argv)
{
    using namespace conef;
    const char *kind = argv[1];
    const bool step = !strcmp(kind, "step");
    const int per = step ? 2 : 3;
    std::vector<int64_t> rows, cols, buckets;
    for (int i = 6; i + per <= argc; i += per) {
        rows.push_back(atoll(argv[i]));
        cols.push_back(atoll(argv[i + 1]));
        if (!step) buckets.push_back(atoll(argv[i + 2]));
    }
    const int rank = atoi(argv[2]), bits = atoi(argv[3]), block = atoi(argv[4]), dtype = atoi(argv[5]), n = (int)rows.size();
    Plan plan;
    const int rc = step ? make_plan(plan, rows.data(), cols.data(), n, rank, bits, block, dtype, 1)
                        : make_sketch_plan(plan, rows.data(), cols.data(), buckets.data(), n, rank, 0.9f, 1, dtype, 1, !strcmp(kind, "columns"));
    if (rc != 0) return 2;
    int chunks = 1;
    for (const MatDesc &d : plan.mats) chunks = d.n_p_chunks > chunks ? d.n_p_chunks : chunks;
    printf("{\"ok\": %d, \"q_joined\": %d, \"err_t_items\": %zu, \"err_rows\": %d, \"norm_back\": %d, \"norm_back_two\": %d, \"csc_rows_p\": %d, "
           "\"one_launch\": %d, \"orth_rows\": %d, \"p_chunks\": %d, \"walk\": %zu, \"row_order\": %zu, \"missed\": [",
           check_plan(plan), plan.q_joined, plan.err_t_items.size(), plan.err_t_items.empty() ? 0 : plan.err_t_items[0].c, plan.norm_back,
           plan.norm_back_two, plan.csc_p_items.empty() ? 0 : plan.csc_p_items[0].c, plan.small_lds > 0, !plan.orth_first.empty(), chunks,
           plan.err_w_items.size(), plan.row_order.size());
    const char *comma = "";
    auto plant = [&](const char *what, auto change) {
        Plan bad = plan;
        change(bad);
        if (check_plan(bad)) printf("%s\"%s\"", comma, what), comma = ", ";
    };
    if (!plan.row_order.empty()) {          // (its last entry is one of a matrix that reads it)
        plant("a row of row_order", [](Plan &p) { p.row_order.back()[0] ^= 1; });
        plant("a bucket of row_order", [](Plan &p) { p.row_order.back()[1] += 1; });
        plant("the length of row_order", [](Plan &p) { p.row_order.pop_back(); });
    }
    if (!plan.orth_first.empty()) {
        plant("an entry of orth_first", [](Plan &p) { p.orth_first.back() += 1; });
        plant("the length of orth_first", [](Plan &p) { p.orth_first.push_back(0); });
    } else {
        plant("orth_first beyond its limits", [](Plan &p) {
            int32_t first = 0;
            for (const MatDesc &d : p.mats) p.orth_first.push_back(first), first += d.n_gram_tiles;
        });
    }
    if (plan.small_lds > 0) plant("small_lds", [](Plan &p) { p.small_lds -= 16; });
    else plant("small_lds of another model", [](Plan &p) { p.small_lds = kSmallLds; });
    printf("]}\n");
    return 0;
}
