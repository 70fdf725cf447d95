// The scoring kernel for rank counts that fill no tiling exactly: more than 8 192 ranks.
#define GD_SCORE_RAGGED 2
#include "score.hip"
