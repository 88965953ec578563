// Which form of the scans a call takes (host only, no device code).  Each form
// gives the same bits; the lines lie where the timings of both forms cross.
#pragma once

namespace comba {

// The rows a scan walks: whole sequences, or their segments in the segmented scans.
struct ScanRows {
  long rows;     // workgroups per head and column slice
  long tokens;   // of all rows
  long chunks;   // of all rows
  long longest;  // chunks of the longest row; 0: not known (packed sequences without host offsets)
};

// Chains (one workgroup each) and, of these, how many are at work on average
// until the longest is done.  Unequal rows leave a few long chains alone on the
// chip for most of the time, however many there are.
inline long scan_chains(const ScanRows& r, int H, int dv) { return r.rows * H * (dv / 32); }
inline long scan_concurrency(const ScanRows& r, int H, int dv) { return r.chunks * H * (dv / 32) / r.longest; }

// Forward scan: whether to move K, Q, the outputs and the saved states as whole
// rows (a quarter of the requests at the address unit, for more LDS traffic and
// latency).  dk = 256 does not fit a CU twice and never takes it.  Gains where
// every CU holds several workgroups whose requests queue.  Time of the direct
// form / of the whole-row form, 256 CUs, H16, stateless and storing:
//  - chains: 1,024 tokens, d128, 384 / 512 / 640 / 768 / 896 / 1,024 chains: 0.97
//    0.97 / 0.98 1.00 / 0.97 0.99 / 1.01 1.02 / 1.02 1.04 / 1.03 1.05.
//  - concurrency (d128, unequal rows of 512 to 4,096 chains): 45: 0.87 0.81, 121:
//    0.87 0.87, 195: 0.95 0.95, 230: 0.96 0.97, 276: 0.99 0.99, 288: 1.02 1.02,
//    336: 1.02 1.03, 496: 1.05 1.05.
//  - chunks partly filled: the direct form repeats the last row, whose lines are
//    there already, the whole-row form does not get shorter.  3,200 chains of four
//    chunks, H4, 256 / 240 / 224 / 200 tokens: 1.02 / 0.99 / 0.98 / 0.96; one
//    chunk of 16 rows 0.94 0.92.
//  - chunk steps per CU, the time over which the longer start-up is spread: full
//    chunks at d64, 6 / 19 / 25 / 50 / 100: 0.97 0.95 0.96 1.02 1.04; at d128 full
//    chunks gain from 8 on (1.08), chunks filled to 7/8 from 40 on (15: 0.97 0.94,
//    30: 0.96 0.98, 40: 0.99 1.01, 54: 1.01 1.01).
//  - longest row not known: the direct form, which loses 10% at most where the
//    other would lose 20%.
inline bool scan_fwd_whole_rows(const ScanRows& r, int H, int dk, int dv, int cus) {
  if (dk > 128 || cus <= 0 || r.longest <= 0) return false;
  if (scan_chains(r, H, dv) < 3L * cus) return false;
  if (4 * scan_concurrency(r, H, dv) < 5L * cus) return false;
  const bool full = 64 * r.tokens >= 63 * 64 * r.chunks;
  if (dk == 128 && full) return true;
  return 8 * r.tokens >= 7 * 64 * r.chunks && r.chunks * H * (dv / 32) >= 40L * cus;
}

// Reverse scan at dk = 128: whether to take the unpadded tiles, with which two
// workgroups fit a CU (their addresses cost 2-5% where only one is there).
// Padded / unpadded, backward from the saved state, H16 d128:
//  - equal rows of 1,024 tokens, 256 / 320 / 448 / 512 / 1,024 chains: 1.00 / 1.12 /
//    1.11 / 1.08 / 1.10; of 64 tokens, 2,048 chains: 1.22.
//  - unequal rows, concurrency 121: 0.97, 195: 0.95, 230: 0.98, 272: 1.04, 276: 0.99,
//    336: 1.08, 438: 1.11.
//  - beside the forward scan of the stateless backward, one workgroup of each form
//    fits a CU with either tiles: 320 / 384 / 448 / 512 / 1,024 chains: 0.96 / 0.97 /
//    1.06 / 1.04 / 1.06; unequal rows, 512 chains and more: 0.99 - 1.04.
//  - longest row not known: by the chains (loses 3-5% at most, gains up to 30%).
// dk = 64 fits a CU twice with padded tiles, whose addresses are simpler (4,096
// tokens, 512 chains: 242.4 us against 246.1); dk = 256 fits once either way.
inline bool scan_bwd_unpadded(const ScanRows& r, int H, int dk, int dv, int cus, bool beside) {
  if (dk != 128 || cus <= 0) return false;
  const long chains = scan_chains(r, H, dv);
  if (beside ? 4 * chains < 7L * cus : chains <= cus) return false;
  return r.longest <= 0 || scan_concurrency(r, H, dv) > cus;
}

}  // namespace comba
