// coop_rounds.h -- how the workgroups of coop.hip share the work and the slots
// of a round: the slices of the matrices and which slot a slice posts in.  No
// HIP types: the layout is made by prep.cpp, and a CPU model of the rounds
// uses the same code.
//
// A round: workgroup i of W posts the slots of its slices i, i + W, ... under
// the round's number, then waits until every slot of the round carries that
// number.  Two sets of slots alternate with the round's number.  That is
// enough if, and only if, every workgroup posts in every round: whoever has
// finished round r has seen everyone's post of r, which each makes after it
// has finished r - 1, so nobody still reads the set of r - 1 when r + 1 is
// posted over it.  A workgroup without a slice of the round's matrix would
// break this (it could fall a round behind unseen, and then wait for a number
// that has been overwritten), so both matrices have at least as many slices
// as there are workgroups, the last ones empty: they post identities.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "schedule.h"

namespace pdhcg {

constexpr int COOP_EPT = 8;          // matrix entries per thread and slice at most

// first of the 8 words of slice s in round `tag`, of slot sets of `slots` slices
constexpr size_t coop_slot(unsigned tag, int slots, int s)
{
    return ((size_t)(tag & 1u) * (size_t)slots + (size_t)s) * 8;
}

struct CoopLayout {
    int threads = 0;                 // of a workgroup
    int full = 0;                    // workgroups of a launch (at most one per CU)
    std::vector<BlkDesc> q, a;       // slices of Q (`full` of them) and of A (`full` at least)
};

// Slices of a CSR: whole rows, at most `threads` of them with at most
// COOP_EPT entries per thread.
std::vector<BlkDesc> coop_slices(int64_t rows, const int64_t* rp, int threads);

// the layout for Q (n rows at qp) and A (m rows at ap) on `cus` CUs; false if
// Q has more slices than that
bool coop_layout(int64_t n, const int64_t* qp, int64_t m, const int64_t* ap, int cus, CoopLayout& L);

}  // namespace pdhcg
