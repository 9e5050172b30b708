// Instances of the fused pass for hash probes whose rows go on together (stage_probe): 4-row items in blocks of up to
// kBigBlock threads.

#include "sdb_fused.h"

namespace sdb {

const void* pick_fused_probe(int ipt, int terminal) {
    if (ipt == 1) { SDB_FUSED_TERMINALS(4, 1, false, kBigBlock, -1) }
    if (ipt == 2) { SDB_FUSED_TERMINALS(4, 2, false, kBigBlock, -1) }
    return nullptr;
}

}  // namespace sdb
