// The launch planner (planner.hpp) on models packed by the library's packer.
#include "planner.hpp"

#include <string>

extern "C" {

// out: level, head, splits, then the tiles of that level and docs_per_block. work as treeens::Work.
int plan_model(int32_t n_trees, const int64_t *tree_offsets, const int32_t *feature, const float *threshold,
               const int32_t *left, const int32_t *right, const float *value, int32_t n_outputs, int32_t n,
               const int32_t *work, const int64_t *n_blocks, int64_t *out) {
    treeens::Packed p;
    std::string err;
    const int rc = treeens::pack_model(n_trees, tree_offsets, feature, threshold, left, right, value, n_outputs, 0, p, err);
    if (rc != treeens::kOk)
        return rc;
    const treeens::PlanFacts f = treeens::plan_facts(p);
    for (int32_t i = 0; i < n; i++) {
        const treeens::Work w = treeens::Work(work[i]);
        const treeens::LaunchShape s = treeens::choose_launch(f, w, n_blocks[i]);
        const treeens::Tiling &t = w == treeens::Work::kTerminal ? f.term : f.walk;
        int64_t *o = out + i * 5;
        o[0] = s.level, o[1] = s.head, o[2] = s.splits, o[3] = t.tiles[s.level], o[4] = p.plan.docs_per_block;
    }
    return 0;
}
}

extern "C" {

// pays[i]: whether documents docs[i] take rule `rule` (0 uniform, 1 terminal, 2 ids stored directly, 3 leaf rows).
int plan_rules(int32_t n_trees, const int64_t *tree_offsets, const int32_t *feature, const float *threshold,
               const int32_t *left, const int32_t *right, const float *value, int32_t n_outputs, int32_t n,
               const int32_t *rule, const int64_t *docs, int32_t *pays) {
    treeens::Packed p;
    std::string err;
    const int rc = treeens::pack_model(n_trees, tree_offsets, feature, threshold, left, right, value, n_outputs, 0, p, err);
    if (rc != treeens::kOk)
        return rc;
    const treeens::PlanFacts f = treeens::plan_facts(p);
    for (int32_t i = 0; i < n; i++)
        pays[i] = rule[i] == 0   ? treeens::uniform_pays(f, docs[i])
                  : rule[i] == 1 ? treeens::term_pays(f, docs[i])
                  : rule[i] == 2 ? treeens::leaves_direct(f, docs[i])
                                 : treeens::rows_pay(f, docs[i]);
    return 0;
}
}
