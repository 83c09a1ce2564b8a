// Dependency records: how the tiles of a launch tell each other that the rows of a down-projection are
// there, in memory that need not be clear when the launch starts.
//
// A record has four 64-bit words per row block: one for each of the producer's (at most two) column tiles,
// a count of the tiles that have seen them all, and a mark.  Producers write the launch's nonce, a number
// that no other launch has, into their words; readers wait for it; the last reader takes it out again, so
// that a replay of the launch, which has the same nonce, finds none.
//   A reader that gives up leaves the nonce in the mark.  The words can keep the nonce of such a launch (its
// producer may have been late, the count short), and a replay would take them for its own producers': with
// the mark set no reader of a launch with this nonce believes them any more.  Its tiles give up at once, visible
// as NaN and in sd_gemm_dep_timeouts, until the memory is cleared or the launch captured anew.
//
// Mem: relaxed loads, stores and adds that all tiles of the launch observe.
#pragma once
#include <stdint.h>
#ifdef __HIPCC__
#define SD_DEP_FN __host__ __device__ __forceinline__
#else
#define SD_DEP_FN inline
#endif

namespace sd {

constexpr int DEP_RECORD = 32;                  // bytes
constexpr int DEP_PRODUCERS = 2;                // column tiles of a producer, at most
constexpr int DEP_COUNT = 2, DEP_GAVE_UP = 3;   // words behind the producers'

// Lane l of a waiting wavefront looks at the word of producer l, the others at the mark (need <= DEP_PRODUCERS)
SD_DEP_FN int dep_record_word(int lane, int need) { return lane < need ? lane : DEP_GAVE_UP; }
// ... and all of its lanes must find this
SD_DEP_FN bool dep_record_ready(int lane, int need, uint64_t v, uint64_t nonce) { return lane < need ? v == nonce : v != nonce; }
SD_DEP_FN bool dep_record_given_up(int lane, int need, uint64_t v, uint64_t nonce) { return lane >= need && v == nonce; }

template <class Mem>
struct DepRecord {
    // producer `tn`: before its last wait for its stores, and after it
    SD_DEP_FN static void open(uint64_t* rec, int tn) {
        if (tn == 0) Mem::store32(reinterpret_cast<int32_t*>(rec + DEP_COUNT), 0);
    }
    SD_DEP_FN static void publish(uint64_t* rec, int tn, uint64_t nonce) { Mem::store64(rec + tn, nonce); }
    // a reader that has waited: its number among the readers, and what the last of them does
    SD_DEP_FN static int leave(uint64_t* rec) { return Mem::add32(reinterpret_cast<int32_t*>(rec + DEP_COUNT), 1); }
    SD_DEP_FN static void clear(uint64_t* rec) {
        for (int i = 0; i < DEP_PRODUCERS; ++i) Mem::store64(rec + i, 0);
    }
    // a reader that has waited long enough
    SD_DEP_FN static void give_up(uint64_t* rec, uint64_t nonce) { Mem::store64(rec + DEP_GAVE_UP, nonce); }
};

}  // namespace sd
