// Prints which kernels a plan sends its passes to, for tests/test_plan_routes.py (host code only; built there with the library's
// plan.cpp).  Arguments: kind (step, rows, columns), rank, bits, block, dtype, then rows and columns of every matrix (and, for the
// sketches, its buckets).
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
    printf("{\"ok\": %d, \"q_joined\": %d, \"err_t_items\": %zu, \"norm_back\": %d, \"norm_back_two\": %d, \"csc_rows_p\": %d}\n",
           check_plan(plan), plan.q_joined, plan.err_t_items.size(), plan.norm_back, plan.norm_back_two,
           plan.csc_p_items.empty() ? 0 : plan.csc_p_items[0].c);
    return 0;
}
