// Answers, on stdout, which launch plan the library takes for the sizes asked for on stdin, one question a line:
//   fwd S heads      -> rows order              order: 0 folded pairs, 1 longest first
//   waves S heads    -> waves of a workgroup of the forward
//   bwd S heads      -> rows, 1 if dK/dV and dQ go out in one launch, order of dK/dV, order of dQ
//   bwdwaves S heads -> waves of a workgroup of the backward
//   lin rows K N     -> tokens and features of a tile
//   window begin end tile tile_rows live -> first row and number of rows of a tile's buffer
//   joint keys queries heads -> for each position of a joint launch the rank of its key tile, or -1 - rank of its query tile
//   f32rows S heads -> head dim 64 in one part: 1 if the forward, and if the backward, brings a workgroup's own rows in once for all waves
//   f32split S heads d -> 1 if the forward, and if the backward, goes to the fp16 matrix instructions
//   divide x d       -> quotient and remainder
//   order rows order -> the order that a shape of that many rows works when asked for `order`
#include "../paper_2407_12117_amd/csrc/launch_plan.h"

#include <cstdio>
#include <cstring>

int main()
{
    char what[16];
    long long a, b, c, d;
    int live;
    while (std::scanf("%15s %lld %lld", what, &a, &b) == 3) {
        if (!std::strcmp(what, "fwd")) {
            const memo::TileChoice &t = memo::fwd_plan(a, b);
            std::printf("%d %d\n", t.rows, t.order);
        } else if (!std::strcmp(what, "waves")) {
            std::printf("%d\n", memo::fwd_plan(a, b).waves);
        } else if (!std::strcmp(what, "bwdwaves")) {
            std::printf("%d\n", memo::bwd_plan(a, b).waves);
        } else if (!std::strcmp(what, "bwd")) {
            const memo::BwdPlan p = memo::bwd_plan(a, b);
            std::printf("%d %d %d %d\n", p.rows, p.joint, p.k_order, p.q_order);
        } else if (!std::strcmp(what, "order")) {
            std::printf("%d\n", memo::tile_order((int)a, (int)b));
        } else if (!std::strcmp(what, "f32rows")) {
            std::printf("%d %d\n", memo::f32_fwd_shares_rows((a + 15) / 16, b), memo::f32_bwd_shares_rows((a + 15) / 16));
        } else if (!std::strcmp(what, "f32split") && std::scanf("%lld", &c) == 1) {
            std::printf("%d\n", memo::f32_splits(a, b, (int)c));
        } else if (!std::strcmp(what, "divide")) {
            const memo::Division r = memo::Divisor(b)((uint32_t)a);
            std::printf("%u %u\n", r.quot, r.rem);
        } else if (!std::strcmp(what, "joint") && std::scanf("%lld", &c) == 1) {
            for (uint32_t pos = 0; pos < a + b; ++pos) {
                const memo::JointSlot s = memo::joint_slot((uint32_t)a, pos);
                std::printf("%d ", s.key ? (int)s.rank : -1 - (int)s.rank);
            }
            std::printf("\n");
        } else if (!std::strcmp(what, "lin") && std::scanf("%lld", &c) == 1) {
            const memo::LinChoice &l = memo::lin_plan(a, (int)b, (int)c);
            std::printf("%d %d\n", l.bm, l.bn);
        } else if (!std::strcmp(what, "window") && std::scanf("%lld %lld %d", &c, &d, &live) == 3) {
            const memo::RowWindow w = memo::row_window(a, b, c, (int)d, live);
            std::printf("%lld %d\n", (long long)w.first, w.rows);
        } else {
            return 1;
        }
    }
    return 0;
}
