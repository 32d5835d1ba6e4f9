// Host check of the rules that choose a kernel by what a list's plan has counted: prints the route of each list given on stdin.
//   segreduce RANK nnz segments tiles distinct common joins pieces       -> walk | pieces
//   mttkrp RANK nnz fibers few-of-C few-of-B longest-slice              -> wave | walk
#include <cstdio>
#include <cstring>

#include "../../paper_2102_05187_amd/csrc/routes.hpp"

int main() {
    char op[32];
    while (scanf("%31s", op) == 1) {
        comet::Schedule sc;
        long rank, nnz, nseg, ntiles, distinct, joins, pieces;
        double common;
        if (!strcmp(op, "segreduce")) {
            if (scanf("%ld %ld %ld %ld %ld %lf %ld %ld", &rank, &nnz, &nseg, &ntiles, &distinct, &common, &joins, &pieces) != 8) return 1;
            sc.nnz = nnz;
            sc.nseg = nseg;
            sc.pieces.ntiles = ntiles;
            sc.pieces.distinct = distinct;
            sc.pieces.common = common;
            sc.pieces.njoins = joins;
            sc.pieces.npieces = pieces;
            printf("%s\n", comet::segreduce_takes_walk(sc, rank) ? "walk" : "pieces");
        } else if (!strcmp(op, "mttkrp")) {
            long few, parent_few, slice;
            if (scanf("%ld %ld %ld %ld %ld %ld", &rank, &nnz, &nseg, &few, &parent_few, &slice) != 6) return 1;
            sc.nnz = nnz;
            sc.nseg = nseg;
            sc.pieces.few = few;
            sc.pieces.parent_few = parent_few;
            sc.max_parent_len = slice;
            printf("%s\n", comet::mttkrp_takes_wave(sc, rank) ? "wave" : "walk");
        } else {
            return 1;
        }
    }
    return 0;
}
